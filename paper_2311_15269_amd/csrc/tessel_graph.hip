// The graph kernel (gfx950): scores repetend candidates of the problems the fast kernel does not take -- any acyclic
// micro-batch graph, up to 32 devices, 64 block types, eight types on a device, windows of 16 micro-batches -- one
// candidate per lane, with the same build as the fast kernel made independent of the number of devices and types.
//
// Two 32-bit masks by device are all that a lane keeps in registers between two blocks: HD = devices whose head may run,
// RD = devices with any type that may run.  Everything indexed by a device or a type sits in LDS, [row][lane]:
//   device record   the order as np bit planes, the entries not yet placed, and one word: symbols that may run (8 bits),
//                   head of the list (one-hot, 8 bits), memory now (signed, 16 bits)
//   type word       next micro-batch, and fields with a guard bit each: occurrences left, and per producer the micro-batches
//                   waiting at the input.  One addition places a block; the type may run iff no field is zero, which
//                   one addition and one compare of the guard bits tell
// One block is placed per step and lane (any order of heads that may run gives the same per-device orders): lowest
// device of HD, else (repair) of RD; there the earliest entry whose type may run.  Three dependent rounds of LDS reads:
// the record; the tables of the (device, symbol); words and records these name.
//
// Bound by the latency of those rounds at the few waves per CU that the LDS holds (a record is np + 2 rows of 256
// bytes per device, a word one row per type), and by VALU issue where there are four waves a SIMD.  Kernel times against the
// general kernel, which looks at every device's head in turn and keeps counters for 64 types in registers: 2^22 candidates of a graph of
// 6 types on three devices, 24 blocks, 3.48 -> 0.708 ms.  LDS decides how many waves hide each other's rounds, so tables are
// as large as the problem, not its limits, and slot states are bytes.
//
// Chains in the sampled spaces (KIND 3 and 4; most wide problems are chains) keep masks by code in registers instead of words by
// type in LDS, as the fast kernel does: two rounds a block instead of three, 40 to 55 % of the LDS, 16-bit times in the
// sweeps.  Against words by type: 200,003 candidates of a pipeline on 16 devices, 256 blocks a window, 0.438 -> 0.255 ms
// (general kernel 34.6); 100,003 of one on 12 devices, 288 blocks, 0.249 -> 0.176 (10.0); 300,007 with six types on each of four
// devices, 96 blocks, 0.205 -> 0.152 (6.9); 3,849 on 15 devices, 360 blocks, 0.275 -> 0.195; 20,725 on 27 devices 0.135 -> 0.086.
//
// Graphs with up to two producers and two consumers a type, small devices and windows (KIND 5) do likewise: a mask by code for either
// producer says whose micro-batch waits, and the two masks and the types that are not used up tell what may run, without a look at any other type's word.
// Two rounds of LDS reads and 60 vector instructions a block instead of three and 105, a third of the LDS, 16-bit times: 2^22 candidates of the K-shape
// (24 blocks on three devices) 497 -> 312 us a call under a tight cap and 769 -> 581 under a wide one, of the diamond at eight
// micro-batches (64 blocks on four) 2,372 -> 899; 64 to 100,003 candidates 0.73 to 0.89 of the time.
//
// The program (block type and micro-batch, 16 bits a block) goes to global memory, [word][slot], a slot per candidate;
// sweeps read it back four words ahead.  A wave owns kGraphSlots slots: candidates that survive the build keep theirs
// until 64 wait, are swept on full waves, and the few whose boundary values have not settled wait again for a longer
// search.  What is open after that goes to the general kernel's list.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>

#include "tessel_common.h"

namespace tessel {

constexpr uint32_t kRow = kWave * 4u;            // one LDS row: a word per lane
constexpr int kTwoWindows = 6;                   // sweeps of the longer search before it goes by two windows
constexpr uint32_t kProgRow = kGraphSlots;       // words of one program word over all slots of a wave

__device__ __forceinline__ void lds_add(uint32_t a, uint32_t v)
{
    __hip_atomic_fetch_add((lds_word *)(uintptr_t)a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// two words in a row, eight-byte aligned
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2 lds_pair;
__device__ __forceinline__ void lds_load2(uint32_t a, uint32_t &x, uint32_t &y)
{
    const u32x2 v = *(const lds_pair *)(uintptr_t)a;
    x = v.x; y = v.y;
}
typedef __attribute__((address_space(3))) uint8_t lds_byte;
__device__ __forceinline__ uint32_t lds_load8(uint32_t a) { return *(const lds_byte *)(uintptr_t)a; }
__device__ __forceinline__ void lds_store8(uint32_t a, uint32_t v) { *(lds_byte *)(uintptr_t)a = (uint8_t)v; }

// the lowest set bit of a mask of up to 64 codes (not 0: any number below 64 then)
__device__ __forceinline__ uint32_t low_bit(uint64_t x)
{
    return min(low_bit((uint32_t)x), low_bit((uint32_t)(x >> 32)) | 32u) & 63u;
}
template <bool W64> struct Codes { typedef uint32_t mask; };
template <> struct Codes<true> { typedef uint64_t mask; };

// KIND: 0 every type has at most one producer and one consumer, 1 any graph, 2 some block sits on several devices; 3 and 4
// chains in the sampled spaces on masks by code, up to 32 and up to 64 codes (GraphTab::codes); 5 such graphs, up to 32 codes.
// NP: bits of a symbol; 0 (with masks by code): one bit, order and entries left in one word.
template <int NP, bool REPAIR, int KIND>
__global__ __launch_bounds__(kWave, KIND >= 3 ? 4 : 1) void eval_graph_kernel(const KParams *__restrict__ Pp, const GraphTab *__restrict__ Gp, uint64_t first,
                                                           uint64_t count, BlockRec *__restrict__ recs, int32_t *__restrict__ code_out,
                                                           int32_t *__restrict__ peak_out, uint64_t *__restrict__ out_list,
                                                           uint32_t *__restrict__ out_count, uint32_t out_cap,
                                                           uint32_t *__restrict__ overflow, uint32_t *slots_all, GraphTurns waves)
{
    extern __shared__ uint32_t lds[];
    // all LDS addresses below are offsets from 0: nothing else of the kernel lies in front of this array
    if (lds_address(lds) != 0u) { if (threadIdx.x == 0) *overflow = 0x100u; return; }
    const KParams &P = *Pp;
    const GraphTab &G = *Gp;
    const bool in_last = blockIdx.x < waves.more;
    uint32_t turns = in_last ? waves.few_last : waves.few_others;
    const int lane = threadIdx.x;
    const uint32_t lane4 = (uint32_t)lane * 4u;
    for (int w = lane; w < G.ntab; w += kWave) lds[w] = G.tab[w];
    const uint32_t sel_row = G.slot_rows, st_row = G.slot_rows + kWave;      // a byte per lane, a byte per slot
#pragma unroll
    for (int j = 0; j < 3; j++) lds_store8(st_row + (uint32_t)(j * kWave + lane), 0u);
    __syncthreads();

    constexpr bool TP = KIND == 2, CODES = KIND >= 3, GRAPH = KIND == 5, CHAIN = KIND == 0 || (CODES && !GRAPH), W64 = KIND == 4;
    const uint32_t cw4 = CHAIN ? 16u : G.code_bytes;             // bytes of one code's table words
    constexpr uint32_t RS = GRAPH ? 3 * kRow : CODES ? (NP == 0 ? 2 : NP == 1 ? 3 : NP + 3) * kRow : (NP + 2) * kRow;      // bytes of one device record
    // rows of end times and device times: 16 bits with masks by code (the host sees that they fit)
    constexpr uint32_t SROW = CODES ? kRow / 2 : kRow;
    const uint32_t lane_s = CODES ? (uint32_t)lane * 2u : lane4;
    auto time_load = [&](uint32_t a) -> uint32_t { return CODES ? lds_load16(a) : lds_load(a); };
    auto time_store = [&](uint32_t a, uint32_t v) { if (CODES) lds_store16(a, v); else lds_store(a, v); };
    const int D = P.D, K = P.K, M = P.M, total = P.total, space = P.space, nwords = G.nwords;
    const uint32_t NR = (uint32_t)P.NR, ADD = G.add, GUARD = G.guard, mushift = (uint32_t)G.mushift;
    const uint32_t rec0 = G.rec + lane4, wrow0 = G.wrow + lane4;
    const int maxout = CHAIN ? 1 : G.maxout, ntp = TP ? G.ntp : 0;
    uint32_t *slots = slots_all + (size_t)blockIdx.x * (size_t)(G.meta + nwords) * kProgRow;
    uint32_t *progs = slots + (size_t)G.meta * kProgRow;
    const uint32_t busy = G.busy;
    const bool idle = __builtin_popcount(busy) < D;
    const bool drop_mem = REPAIR && peak_out == nullptr;         // a rejected candidate's peak is that of the whole window

    int best = INT_MAX;
    uint64_t best_idx = 0;
    uint32_t cnt[kNumStatus];
#pragma unroll
    for (int s = 0; s < kNumStatus; s++) cnt[s] = 0;
    uint32_t nev = 0, nretry = 0;

    auto rank_in = [&](uint64_t m) -> uint32_t {
        return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    };
    // (table words with a uniform index come from the LDS copy too)
    auto uniform_word = [&](uint32_t a) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_load(a)); };
    auto types_on = [&](int d) -> uint32_t { return uniform_word(G.dev + (uint32_t)d * 4u); };
    auto ready = [&](uint32_t w) -> bool { return ((w + ADD) & GUARD) == GUARD; };
    // The first 64 slots in state `cls`, one per lane (fewer: the other lanes get some slot of the wave); how many there
    // are.  `take` false: only counts.
    auto slots_in = [&](uint32_t cls, bool take, uint32_t &mine) -> uint32_t {
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const bool in = lds_load8(st_row + (uint32_t)(j * kWave + lane)) == cls;
            const uint64_t m = __ballot(in);
            if (take && in) {
                const uint32_t r = n + rank_in(m);
                if (r < (uint32_t)kWave) lds_store8(sel_row + r, (uint32_t)(j * kWave + lane));
            }
            n += (uint32_t)__builtin_popcountll(m);
        }
        if (take) { __syncthreads(); mine = lds_load8(sel_row + (uint32_t)lane); __syncthreads(); }
        return n;
    };

    // ---------------------------------------------------------------- chains on masks by code
    // Decode and build of 64 candidates (KIND 3 and 4).  A type that gets a micro-batch may run unless its entries are used up,
    // whatever else is true of it: masks by code in registers (R types that may run, HM heads, X used up) say so without a look
    // at the consumer, whose record gets its micro-batch by an atomic nobody waits for.  Two dependent rounds of LDS reads a
    // block (record, table words of the code) where the words by type need three, and less LDS: a device's types have no rows of
    // their own.
    auto build_codes = [&](uint32_t ka, uint32_t kb, bool valid, uint32_t *prog, int &status, int &worst, bool &whole) {
        typedef typename Codes<W64>::mask mask_t;
        constexpr int NB = NP == 0 ? 1 : NP;                     // bits of a symbol
        constexpr uint32_t TS = W64 ? 256u : 128u;               // bytes of one table word over all codes
        constexpr uint32_t DEV = (1u << (1 << NB)) - 1u;         // the codes of one device
        constexpr bool ONE = NP <= 1;                            // waiting micro-batches, leads and memory in one word
        constexpr uint32_t row_alive = NP == 0 ? 0u : NB, row_w = NP == 0 ? 1u : NB + 1, row_l = ONE ? row_w : NB + 2;
        mask_t R = 0, HM = 0, X = 0;
        for (int d = 0; d < D; d++) {
            lds_store(rec0 + (uint32_t)d * RS + row_w * kRow, 0u);
            if (!ONE) lds_store(rec0 + (uint32_t)d * RS + row_l * kRow, 0u);
        }
        // ---- leads, every chain from its last type to its first; a type's waiting micro-batches are what its producer's lead
        // is ahead (no producer: more than it has blocks)
        {
            uint32_t lead = 0, at = ~0u, word = 0;
            for (int k = 0; k < K; k++) {
                const uint32_t c0 = G.links[k][0], c1 = G.links[k][1], c2 = G.links[k][2];
                const bool last = c0 >> 25 & 1u, first_type = c0 >> 26 & 1u;
                const uint32_t before = lead, e = c0 >> 16 & 255u;
                if (P.has_fixed) lead = c2 >> 28;
                else {
                    uint32_t stepped = 0;
                    if (c0 >> 24 & 1u) {
                        const uint32_t wi = (kDrawLeadBase + e) >> 1;
                        if (wi != at) { word = stream_word(ka, kb, wi); at = wi; }
                        stepped = ((e & 1u) ? word >> 16 : word & 0xFFFFu) < P.step_q16 ? 1u : 0u;
                    }
                    lead = last ? 0u : min(NR - 1u, lead + stepped);
                }
                if (!last) {
                    // the consumer, the entry before: its waiting micro-batches
                    const uint32_t b0 = G.links[k - 1][0], b1 = G.links[k - 1][1], waits = lead - before;
                    lds_add((b0 & 0xFFFFu) + lane4, waits << (b1 & 31u));
                    R |= (mask_t)min(waits, 1u) << (b1 >> 8 & 63u);
                }
                if (first_type) {
                    lds_add((c0 & 0xFFFFu) + lane4, (NR + 1u) << (c1 & 31u));
                    R |= (mask_t)1u << (c1 >> 8 & 63u);
                }
                lds_add((c0 & 0xFFFFu) + (row_l - row_w) * kRow + lane4, (lead << (c1 >> 16 & 31u)) + lead * G.links[k][3]);
            }
        }
        // ---- orders, by device
        for (int d = 0; d < D; d++) {
            const uint32_t ntd = (uint32_t)P.ntd[d], n = ntd * NR;
            Planes<NB> o;
            sampled_order<NB>(ka, kb, d, ntd, NR, o);
            const uint32_t ra = rec0 + (uint32_t)d * RS, alive = n >= 32u ? 0xFFFFFFFFu : (1u << n) - 1u;
            if (NP == 0) lds_store(ra, o.p0 | alive << 16);
            else {
                lds_store(ra, o.p0);
                if (NB > 1) lds_store(ra + kRow, o.p1);
                if (NB > 2) lds_store(ra + 2 * kRow, o.p2);
                lds_store(ra + row_alive * kRow, alive);
            }
            const uint32_t y0 = (o.p0 & 1u) | (NB > 1 ? (o.p1 & 1u) << 1 : 0u) | (NB > 2 ? (o.p2 & 1u) << 2 : 0u);
            if (n) HM |= (mask_t)1u << (((uint32_t)d << NB) + y0);
        }
        // ---- blocks in an executable sequence
        bool building = REPAIR || valid;
        const uint32_t last_dev = ((uint32_t)D - 1u) << NB;
        auto step = [&]() -> uint32_t {
            const mask_t hm = R & HM, sel = hm ? hm : (REPAIR ? R : (mask_t)0);
            if (!REPAIR && building && sel == 0) { status = kDeadlock; building = false; }
            // the device's first code
            uint32_t d0 = low_bit(sel) & ~((1u << NB) - 1u);
            d0 = REPAIR ? min(d0, last_dev) : building ? d0 : 0u;
            TESSEL_PIN(d0);
            const uint32_t ra = __umul24(d0, RS >> NB) + rec0;
            const uint32_t p0 = lds_load(ra), p1 = NB > 1 ? lds_load(ra + kRow) : 0u, p2 = NB > 2 ? lds_load(ra + 2 * kRow) : 0u;
            const uint32_t alive = NP == 0 ? p0 >> 16 : lds_load(ra + row_alive * kRow);
            const uint32_t w = lds_load(ra + row_w * kRow), l = ONE ? w : lds_load(ra + row_l * kRow);
            // earliest entry whose type may run: a multiplexer keyed by the planes.  (A device picked for its head: the head.)
            const uint32_t may = W64 ? (d0 & 32u ? (uint32_t)((uint64_t)R >> 32) : (uint32_t)R) >> (d0 & 31u) : (uint32_t)R >> d0;
            auto runs = [&](int y) -> uint32_t { return (uint32_t)__builtin_amdgcn_sbfe((int)may, y, 1); };
            uint32_t gate;
            if (NB == 1) gate = bfi(p0, runs(1), runs(0));
            else {
                gate = bfi(p1, bfi(p0, runs(3), runs(2)), bfi(p0, runs(1), runs(0)));
                if (NB > 2) gate = bfi(p2, bfi(p1, bfi(p0, runs(7), runs(6)), bfi(p0, runs(5), runs(4))), gate);
            }
            const uint32_t p = low_bit(alive & gate);
            // its symbol as all-or-nothing masks, its code
            const uint32_t ly = (uint32_t)__builtin_amdgcn_sbfe((int)p0, p, 1), hy = NB > 1 ? (uint32_t)__builtin_amdgcn_sbfe((int)p1, p, 1) : 0u;
            const uint32_t zy = NB > 2 ? (uint32_t)__builtin_amdgcn_sbfe((int)p2, p, 1) : 0u;
            const uint32_t y = (ly & 1u) | (hy & 2u) | (zy & 4u), c = d0 + y, ca = c << 2;
            const uint32_t t_add = lds_load(ca), t_next = lds_load(ca + TS), t_at = lds_load(ca + 2 * TS), t_inc = lds_load(ca + 3 * TS);
            const uint32_t t_mem = ONE ? 0u : lds_load(ca + 4 * TS), t_next_hi = W64 ? lds_load(ca + 5 * TS) : 0u;
            // (worked out while the table words are on their way) the entry out, the device's new head.  (A device that is empty
            // now gets a meaningless bit, and a harmless one: its types are used up, and R holds no such type.)
            const uint32_t left = alive & ~(1u << p), q = low_bit(left);
            uint32_t y2 = __builtin_amdgcn_ubfe(p0, q, 1);
            if (NB > 1) y2 |= __builtin_amdgcn_ubfe(p1, q, 1) << 1;
            if (NB > 2) y2 |= __builtin_amdgcn_ubfe(p2, q, 1) << 2;
            const mask_t hm_new = (HM & ~((mask_t)DEV << d0)) | (mask_t)1u << (d0 + y2);
            uint32_t rest = left & ~(p0 ^ ly);                   // entries of the type that are left
            if (NB > 1) rest &= ~(p1 ^ hy);
            if (NB > 2) rest &= ~(p2 ^ zy);
            const uint32_t at_w = NP == 3 ? 4u * y : NP == 2 ? 5u * y : ly & 5u;
            const uint32_t more = __builtin_amdgcn_ubfe(w, at_w, NP == 3 ? 4 : 5);
            const uint32_t lead = ONE ? __builtin_amdgcn_ubfe(l, (ly & 4u) | 10u, 4) : NP == 2 ? __builtin_amdgcn_ubfe(l, 4u * y, 4) : __builtin_amdgcn_ubfe(l, 3u * y, 3);
            const mask_t onec = (mask_t)1u << c;
            const bool used_up = rest == 0, stalled = used_up | (more < 2u);
            const mask_t x_new = X | (used_up ? onec : (mask_t)0);
            const mask_t next = W64 ? (mask_t)(t_next | (uint64_t)t_next_hi << 32) : (mask_t)t_next;
            const mask_t r_new = (R & ~(stalled ? onec : (mask_t)0)) | (next & ~x_new);
            const uint32_t w_new = w + t_add, l_new = ONE ? w_new : l + t_mem;
            uint32_t entry = 0;
            if (REPAIR || building) {
                if (NP == 0) lds_store(ra, p0 & ~(0x10000u << p)); else lds_store(ra + row_alive * kRow, left);
                lds_store(ra + row_w * kRow, w_new);
                if (!ONE) lds_store(ra + row_l * kRow, l_new);
                lds_add((t_at & 0xFFFFu) + lane4, t_inc);        // (no consumer: 0 to its own record)
                worst = max(worst, (int)l_new >> (ONE ? 18 : NP == 2 ? 16 : 24));
                R = r_new; X = x_new; HM = hm_new;
                entry = ((lead - (uint32_t)__builtin_popcount(rest)) << 9) + (t_at >> 16);       // 8 type, micro-batch << 9: lead + N_R - 1 - entries left
            }
            return entry;
        };
        const int full = total / 2;
        whole = true;
        for (int wi = 0; wi < full; wi++) {
            const uint32_t e0 = step(), e1 = step();
            prog[(size_t)wi * kProgRow] = e0 | e1 << 16;
            if (!REPAIR || (wi & 7) == 7) {
                if (__builtin_expect((wi & 7) == 7 && turns != 0, 0)) take_turn(turns);
                const bool going = valid && (REPAIR ? !(drop_mem && worst > M) : building);
                if (__ballot(going) == 0) { whole = false; break; }
            }
        }
        if (whole && (total & 1)) prog[(size_t)full * kProgRow] = step();
    };

    // ---------------------------------------------------------------- graphs on masks by code
    // The same with two producers and two consumers a type (KIND 5): W0 and W1 types for which a micro-batch of the first, of the second
    // producer waits (of one that is not there: always), so that W0 & W1 & ~X may run.  A device's record: order and entries left; the
    // waiting micro-batches, five bits a producer; leads and memory.
    auto build_graph = [&](uint32_t ka, uint32_t kb, bool valid, uint32_t *prog, int &status, int &worst, bool &whole) {
        constexpr uint32_t TS = 128u;                            // bytes of one table word over all codes
        uint32_t W0 = G.free0, W1 = G.free1, HM = 0, X = 0;
        // ---- leads, four bits a type, consumers before producers
        uint64_t leads = 0;
        if (P.has_fixed)
            for (int g = 0; g < K; g++) leads |= (uint64_t)P.fixed[g] << (4 * g);
        else {
            uint32_t lead = 0, at = ~0u, word = 0;
            for (int k = 0; k < G.nlead; k++) {
                const uint32_t E = G.lead_edge[k], src = E & 255u, dst = E >> 8 & 255u, e = E >> 16 & 255u;
                if (E >> 25 & 1u) lead = 0;
                uint32_t stepped = 0;
                if (E >> 24 & 1u) {
                    const uint32_t wi = (kDrawLeadBase + e) >> 1;
                    if (wi != at) { word = stream_word(ka, kb, wi); at = wi; }
                    stepped = ((e & 1u) ? word >> 16 : word & 0xFFFFu) < P.step_q16 ? 1u : 0u;
                }
                lead = max(lead, ((uint32_t)(leads >> (4 * dst)) & 15u) + stepped);
                if (E >> 26 & 1u) { lead = min(NR - 1u, lead); leads |= (uint64_t)lead << (4 * src); }
            }
        }
        auto lead_of = [&](uint32_t g) -> uint32_t { return (uint32_t)(leads >> (4 * g)) & 15u; };
        // ---- records
        for (int d = 0; d < D; d++) {
            const uint32_t ntd = (uint32_t)P.ntd[d], n = ntd * NR;
            Planes<1> o;
            sampled_order<1>(ka, kb, d, ntd, NR, o);
            const uint32_t ra = rec0 + (uint32_t)d * RS;
            lds_store(ra, o.p0 | ((1u << n) - 1u) << 16);        // (16 entries at most)
            lds_store(ra + kRow, G.waits[d]);
            lds_store(ra + 2 * kRow, 0u);
            if (n) HM |= 1u << (2u * (uint32_t)d + (o.p0 & 1u));
        }
        for (int g = 0; g < K; g++)
            lds_add(G.links[g][0] + kRow + lane4, (lead_of((uint32_t)g) << (G.links[g][1] & 31u)) + lead_of((uint32_t)g) * G.links[g][3]);
        for (int k = 0; k < G.nedge; k++) {
            const uint32_t E = G.edge[k], dst = E >> 8 & 255u, ahead = lead_of(E & 255u) - lead_of(dst), bit = min(ahead, 1u) << (G.links[dst][1] >> 8 & 31u);
            lds_add(G.links[dst][0] + lane4, ahead << (E >> 16 & 31u));
            if (E >> 24) W1 |= bit; else W0 |= bit;
        }
        // ---- blocks in an executable sequence
        bool building = REPAIR || valid;
        const uint32_t last_dev = ((uint32_t)D - 1u) << 1;
        auto step = [&]() -> uint32_t {
            const uint32_t R = __builtin_amdgcn_bitop3_b32(W0, W1, X, 0x40), hm = R & HM, sel = hm ? hm : (REPAIR ? R : 0u);        // a & b & ~c
            if (!REPAIR && building && sel == 0) { status = kDeadlock; building = false; }
            uint32_t d0 = low_bit(sel) & ~1u;                    // the device's first code
            d0 = REPAIR ? min(d0, last_dev) : building ? d0 : 0u;
            TESSEL_PIN(d0);
            const uint32_t ra = __umul24(d0, RS / 2) + rec0;
            const uint32_t p0 = lds_load(ra), w = lds_load(ra + kRow), l = lds_load(ra + 2 * kRow), alive = p0 >> 16;
            const uint32_t may = R >> d0;
            const uint32_t gate = bfi(p0, (uint32_t)__builtin_amdgcn_sbfe((int)may, 1, 1), (uint32_t)__builtin_amdgcn_sbfe((int)may, 0, 1));
            const uint32_t p = low_bit(alive & gate), ly = (uint32_t)__builtin_amdgcn_sbfe((int)p0, p, 1), c = d0 - ly, ca = c << 2;
            const uint32_t t_add = lds_load(ca), t_mem = lds_load(ca + TS), t_next0 = lds_load(ca + 2 * TS), t_next1 = lds_load(ca + 3 * TS);
            const uint32_t t_at = lds_load(ca + 4 * TS), t_inc = lds_load(ca + 5 * TS), t_at2 = lds_load(ca + 6 * TS), t_inc2 = lds_load(ca + 7 * TS);
            // (worked out while the table words are on their way)
            const uint32_t left = alive & ~(1u << p), q = low_bit(left), y2 = __builtin_amdgcn_ubfe(p0, q, 1);
            const uint32_t hm_new = (HM & ~(3u << d0)) | 1u << (d0 + y2), rest = left & ~(p0 ^ ly);
            const uint32_t waits = w >> (ly & 10u), lead = __builtin_amdgcn_ubfe(l, ly & 4u, 4), onec = 1u << c;
            const uint32_t w_new = w + t_add, l_new = l + t_mem;
            uint32_t entry = 0;
            if (REPAIR || building) {
                lds_store(ra, p0 & ~(0x10000u << p));
                lds_store(ra + kRow, w_new);
                lds_store(ra + 2 * kRow, l_new);
                lds_add((t_at & 0xFFFFu) + lane4, t_inc);        // (no such consumer: 0 to its own record)
                lds_add(t_at2 + lane4, t_inc2);
                worst = max(worst, (int)l_new >> 16);
                W0 = (W0 & ~(waits & 30u ? 0u : onec)) | t_next0;
                W1 = (W1 & ~(waits & (30u << 5) ? 0u : onec)) | t_next1;
                X |= rest == 0 ? onec : 0u;
                HM = hm_new;
                entry = ((lead - (uint32_t)__builtin_popcount(rest)) << 9) + (t_at >> 16);       // 8 type, micro-batch << 9
            }
            return entry;
        };
        const int full = total / 2;
        whole = true;
        for (int wi = 0; wi < full; wi++) {
            const uint32_t e0 = step(), e1 = step();
            prog[(size_t)wi * kProgRow] = e0 | e1 << 16;
            if (!REPAIR || (wi & 7) == 7) {
                if (__builtin_expect((wi & 7) == 7 && turns != 0, 0)) take_turn(turns);
                const bool going = valid && (REPAIR ? !(drop_mem && worst > M) : building);
                if (__ballot(going) == 0) { whole = false; break; }
            }
        }
        if (whole && (total & 1)) prog[(size_t)full * kProgRow] = step();
    };

    // ---------------------------------------------------------------- build: 64 new candidates
    auto build = [&](uint64_t idx, bool valid) {
        uint32_t slot = 0;
        lds_store8(sel_row + (uint32_t)lane, (uint32_t)lane);
        __syncthreads();
        slots_in(0u, true, slot);                                // (always 64 or more free: see kGraphSlots)
        uint32_t *prog = progs + slot;
        int status = kOk;
        uint32_t ka = 0, kb = 0;
        uint64_t rest = idx;
        const bool sampled = space == kSampledStrict || space == kSampledRepair;
        if (sampled) ka = stream_keys(P.seed, idx, kb);
        int worst = INT_MIN;
        bool any = true, whole = true;
        if constexpr (GRAPH) build_graph(ka, kb, valid, prog, status, worst, whole);
        else if constexpr (CODES) build_codes(ka, kb, valid, prog, status, worst, whole);
        else {
        lds_store(G.trash + lane4, 0u);
        // ---- leads, by type
        for (int g = 0; g < K; g++) {
            uint32_t lead = 0;
            if (sampled && P.has_fixed) lead = P.fixed[g];
            lds_store(wrow0 + (uint32_t)g * kRow, uniform_word(G.init + (uint32_t)g * 4u) + (lead << mushift));
        }
        if (sampled && !P.has_fixed) {
            // consumers before producers: a type's lead is the largest (consumer's lead + step) over its dependencies
            uint32_t lead = 0, before = ~0u, before_lead = 0, at = ~0u, word = 0;
            for (int k = 0; k < G.nlead; k++) {
                const uint32_t E = (uint32_t)__builtin_amdgcn_readfirstlane((int)G.lead_edge[k]);
                const uint32_t src = E & 255u, dst = (E >> 8) & 255u, e = (E >> 16) & 255u;
                if (E >> 25 & 1u) lead = 0;
                const uint32_t ld = dst == before ? before_lead : lds_load(wrow0 + dst * kRow) >> mushift;
                uint32_t step = 0;
                if (E >> 24 & 1u) {
                    const uint32_t wi = (kDrawLeadBase + e) >> 1;
                    if (wi != at) { word = stream_word(ka, kb, wi); at = wi; }
                    const uint32_t u = (e & 1u) ? word >> 16 : word & 0xFFFFu;
                    step = u < P.step_q16 ? 1u : 0u;
                }
                lead = max(lead, ld + step);
                if (E >> 26 & 1u) {
                    lead = min(NR - 1u, lead);
                    lds_store(wrow0 + src * kRow, uniform_word(G.init + src * 4u) + (lead << mushift));
                    before = src; before_lead = lead;
                }
            }
        }
        // ---- orders, by device
        bool dup = false, tpm = false;
        for (int d = 0; d < D; d++) {
            const uint32_t ntd = types_on(d), n = ntd * NR;
            Planes<NP> o;
            if (sampled) sampled_order<NP>(ka, kb, d, ntd, NR, o);
            else if (space == kCanonical) {
                o.clear();
                const uint32_t B = NR + 1;
                uint64_t r = rest % P.cdev[d];
                rest /= P.cdev[d];
                uint32_t c0 = ntd > 0 ? NR : 0u, c1 = ntd > 1 ? NR : 0u, c2 = ntd > 2 ? NR : 0u, c3 = ntd > 3 ? NR : 0u;
                for (uint32_t pos = 0; pos < n; pos++) {
                    bool chosen = false;
                    uint32_t y = 0;
                    auto look = [&](uint32_t &c, uint32_t sym) {
                        if (chosen || c == 0) return;
                        c--;
                        const uint64_t w = P.wtab[((c0 * B + c1) * B + c2) * B + c3];
                        if (r < w) { y = sym; chosen = true; } else { r -= w; c++; }
                    };
                    look(c0, 0u); look(c1, 1u);
                    if (NP > 1) { look(c2, 2u); look(c3, 3u); }
                    o.put(y, pos);
                }
            } else {
                o.clear();
                uint32_t r = (uint32_t)(rest % P.cdev[d]);
                rest /= P.cdev[d];
                uint64_t list = P.init_list[d];
                uint32_t firstlab = 0xFFFFFFFFu, seen = 0;
                for (uint32_t pos = 0; pos < n; pos++) {
                    const uint32_t f = P.fact[n - 1 - pos];
                    const uint32_t digit = r / f;
                    r -= digit * f;
                    const uint32_t code = (uint32_t)(list >> (5u * digit)) & 31u;
                    const uint64_t low = list & ((1ull << (5u * digit)) - 1ull);
                    list = low | (((list >> (5u * digit)) >> 5) << (5u * digit));
                    const uint32_t y = code >> 3, lab = code & 7u;
                    o.put(y, pos);
                    const uint32_t fl = byte_of(firstlab, y), sc = byte_of(seen, y);
                    if (fl == 0xFFu) firstlab = (firstlab & ~(0xFFu << (8u * y))) | (lab << (8u * y));
                    else {
                        uint32_t want = fl + sc;                 // labels continue cyclically (Property 1)
                        if (want >= NR) want -= NR;
                        if (lab != want) dup = true;
                    }
                    seen += 1u << (8u * y);
                }
                for (uint32_t y = 0; y < ntd; y++) {
                    const uint32_t g = uniform_word((((uint32_t)d << NP) + y) * cw4) & 63u;
                    const uint32_t fl = byte_of(firstlab, y), a = wrow0 + g * kRow;
                    if ((uint32_t)__builtin_ctz(P.mask_type[g]) == (uint32_t)d) lds_store(a, uniform_word(G.init + (uint32_t)g * 4u) + (fl << mushift));
                    else if (lds_load(a) >> mushift != fl) tpm = true;
                }
            }
            const uint32_t ra = rec0 + (uint32_t)d * RS;
            lds_store(ra, o.p0);
            if (NP > 1) lds_store(ra + kRow, o.p1);
            if (NP > 2) lds_store(ra + 2 * kRow, o.p2);
            const uint32_t alive = n >= 32u ? 0xFFFFFFFFu : (1u << n) - 1u;
            const uint32_t y0 = (o.p0 & 1u) | (NP > 1 ? (o.p1 & 1u) << 1 : 0u) | (NP > 2 ? (o.p2 & 1u) << 2 : 0u);
            lds_store(ra + NP * kRow, alive);
            lds_store(ra + (NP + 1) * kRow, n ? 1u << (8u + y0) : 0u);
        }
        if (space == kCanonical) {
            const int8_t *row = P.leadtab + rest * (uint64_t)K;
            for (int g = 0; g < K; g++) lds_store(wrow0 + (uint32_t)g * kRow, uniform_word(G.init + (uint32_t)g * 4u) + ((uint32_t)row[g] << mushift));
        }
        // ---- micro-batches waiting at every input: what the last window's producer is ahead of its consumer
        bool prop2 = false;
        for (int k = 0; k < G.nedge; k++) {
            const uint32_t E = (uint32_t)__builtin_amdgcn_readfirstlane((int)G.edge[k]);
            const uint32_t a = wrow0 + (E & 255u) * kRow, b = wrow0 + ((E >> 8) & 255u) * kRow;
            const uint32_t ls = lds_load(a) >> mushift, ld = lds_load(b) >> mushift;
            if (ls < ld) prop2 = true;
            else lds_add(b, (ls - ld) << (E >> 16));
        }
        if (space == kFactorial) status = dup ? kDup : tpm ? kTpMismatch : prop2 ? kProp2 : kOk;
        // (exhaustive spaces: often none of a wave's candidates is left here, or after a few blocks)
        any = REPAIR || __ballot(valid && status == kOk) != 0;
        // ---- what may run, memory at the window entry (type i has handled micro-batches 0 .. lead - 1), heads
        uint32_t RD = 0, HD = 0;
        uint64_t hcnt = 0;                                       // TP: devices a type heads, six bits a type
        uint32_t rtp = 0;                                        // TP: such types that may run
        for (int d = 0; any && d < D; d++) {
            const uint32_t ra = rec0 + (uint32_t)d * RS + (NP + 1) * kRow;
            uint32_t runs = 0;
            int mem = 0;
            const uint32_t head = lds_load(ra);
            const int ntd = (int)types_on(d);
            for (int y = 0; y < ntd; y++) {
                const uint32_t T0 = uniform_word((((uint32_t)d << NP) + (uint32_t)y) * cw4);
                const uint32_t w = lds_load((T0 & 0xFF00u) + lane4);
                const bool ok = ready(w);
                runs |= (ok ? 1u : 0u) << y;
                mem += ((int)T0 >> 16) * (int)(w >> mushift);
                if (TP && (T0 & 64u)) {
                    const uint32_t inf = uniform_word(G.tpi + (T0 & 63u) * 4u);
                    if (head >> (8 + y) & 1u) hcnt += 1ull << (inf & 63u);
                    rtp |= ok ? 1u << ((inf & 63u) / 6u) : 0u;
                }
            }
            const uint32_t smask = TP ? uniform_word(G.smask + (uint32_t)d * 4u) : 0xFFu;
            lds_store(ra, runs | head | ((uint32_t)mem << 16));
            RD |= (runs ? 1u : 0u) << d;
            HD |= (runs & (head >> 8) & smask ? 1u : 0u) << d;
        }
        // ---- blocks in an executable sequence
        bool building = REPAIR || (valid && status == kOk);
        const uint32_t dlast = (uint32_t)D - 1u;
        // the head of a device list changed: TP types it left or reached
        auto head_moved = [&](uint32_t code0, uint32_t from, uint32_t to) {
            if (from == to) return;
            if (from) {
                const uint32_t T = lds_load((code0 | (uint32_t)__builtin_ctz(from)) * cw4);
                if (T & 64u) hcnt -= 1ull << (lds_load(G.tpi + (T & 63u) * 4u) & 63u);
            }
            if (to) {
                const uint32_t T = lds_load((code0 | (uint32_t)__builtin_ctz(to)) * cw4);
                if (T & 64u) hcnt += 1ull << (lds_load(G.tpi + (T & 63u) * 4u) & 63u);
            }
        };
        auto step = [&]() -> uint32_t {
            uint32_t hd = HD;
            if (TP)
                for (int i = 0; i < ntp; i++) {
                    // a type on several devices is a head that may run when it heads all of them; placed from its lowest
                    const uint32_t inf = uniform_word(G.tpi + (kMaxKW + (uint32_t)i) * 4u);
                    const bool full = ((uint32_t)(hcnt >> (6 * i)) & 63u) == inf >> 16;
                    hd |= full && (rtp >> i & 1u) ? 1u << ((inf >> 8) & 31u) : 0u;
                }
            const uint32_t sel = hd ? hd : (REPAIR ? RD : 0u);
            if (!REPAIR && building && sel == 0) { status = kDeadlock; building = false; }
            const uint32_t d = REPAIR ? min(low_bit(sel) & 31u, dlast) : building ? low_bit(sel) & 31u : 0u;
            const uint32_t ra = d * RS + rec0;
            const uint32_t p0 = lds_load(ra), p1 = NP > 1 ? lds_load(ra + kRow) : 0u, p2 = NP > 2 ? lds_load(ra + 2 * kRow) : 0u;
            const uint32_t alive = lds_load(ra + NP * kRow), rhm = lds_load(ra + (NP + 1) * kRow);
            // earliest entry whose type may run: a multiplexer keyed by the planes.  (A device picked for its head: the head.)
            auto runs = [&](int y) -> uint32_t { return (uint32_t)__builtin_amdgcn_sbfe((int)rhm, y, 1); };
            uint32_t gate;
            if (NP == 1) gate = bfi(p0, runs(1), runs(0));
            else {
                gate = bfi(p1, bfi(p0, runs(3), runs(2)), bfi(p0, runs(1), runs(0)));
                if (NP > 2) gate = bfi(p2, bfi(p1, bfi(p0, runs(7), runs(6)), bfi(p0, runs(5), runs(4))), gate);
            }
            const uint32_t p = low_bit(alive & gate);
            auto symbol = [&](uint32_t pos) -> uint32_t {
                uint32_t y = __builtin_amdgcn_ubfe(p0, pos, 1);
                if (NP > 1) y |= __builtin_amdgcn_ubfe(p1, pos, 1) << 1;
                if (NP > 2) y |= __builtin_amdgcn_ubfe(p2, pos, 1) << 2;
                return y;
            };
            const uint32_t y = symbol(p), code0 = d << NP, ca = CHAIN ? (code0 | y) << 4 : __umul24(code0 | y, cw4);
            uint32_t T0, T1, C0, C1;
            lds_load2(ca, T0, T1); lds_load2(ca + 8u, C0, C1);
            uint32_t E0 = 0, E1 = 0;
            if (KIND == 1 && maxout > 1) lds_load2(ca + 16u, E0, E1);
            // (worked out while the table words are on their way)
            const uint32_t alive2 = alive & ~(1u << p);
            uint32_t head2 = 256u << symbol(low_bit(alive2));
            TESSEL_PIN(head2);
            head2 = alive2 ? head2 : 0u;
            const uint32_t wa = (T0 & 0xFF00u) + lane4;
            uint32_t cwa = (C0 & 0xFF00u) + lane4, cra = (C0 >> 16) + lane4;
            uint32_t w = lds_load(wa), wc = lds_load(cwa), rc = lds_load(cra);
            // (a second consumer in the same rounds; what the first changes on its device is passed on in registers)
            uint32_t wd = 0, rd = 0;
            if (KIND == 1 && maxout > 1) { wd = lds_load((E0 & 0xFF00u) + lane4); rd = lds_load((E0 >> 16) + lane4); }
            const uint32_t w2 = w + T1;
            const bool again = ready(w2);
            const uint32_t onec = 1u << y;
            uint32_t rhm2 = ((rhm + (T0 & 0xFFFF0000u)) & 0xFFFF0000u) | (rhm & 0xFFu & ~onec) | (again ? onec : 0u) | head2;
            uint32_t entry = 0;
            if (REPAIR || building) {
                worst = max(worst, (int)rhm2 >> 16);
                lds_store(ra + NP * kRow, alive2);
                lds_store(wa, w2);
                lds_store(ra + (NP + 1) * kRow, rhm2);
                const uint32_t smask = TP ? lds_load(G.smask + (d << 2)) : 0xFFu;
                const uint32_t oned = 1u << d;
                RD = rhm2 & 0xFFu ? RD | oned : RD & ~oned;
                HD = rhm2 & (rhm2 >> 8) & smask ? HD | oned : HD & ~oned;
                if (TP) {
                    head_moved(code0, rhm >> 8 & 0xFFu, head2 >> 8);
                    if (T0 & 64u) {
                        // the block's earliest entry on its other devices
                        const uint32_t g = T0 & 63u, inf = lds_load(G.tpi + g * 4u), i = (inf & 63u) / 6u;
                        rtp = again ? rtp | 1u << i : rtp & ~(1u << i);
                        for (uint32_t others = lds_load(G.tpm + g * 4u) & ~oned; others; others &= others - 1u) {
                            const uint32_t dd = (uint32_t)__builtin_ctz(others), rq = dd * RS + rec0;
                            const uint32_t q0 = lds_load(rq), q1 = NP > 1 ? lds_load(rq + kRow) : 0u, q2 = NP > 2 ? lds_load(rq + 2 * kRow) : 0u;
                            const uint32_t qa = lds_load(rq + NP * kRow), qr = lds_load(rq + (NP + 1) * kRow);
                            const uint32_t ys = lds_load(G.tps + (i * 32u + dd) * 4u);
                            uint32_t same = qa & (ys & 1u ? q0 : ~q0);
                            if (NP > 1) same &= ys & 2u ? q1 : ~q1;
                            if (NP > 2) same &= ys & 4u ? q2 : ~q2;
                            const uint32_t left = qa & ~(same & (0u - same));
                            const uint32_t ph = low_bit(left);
                            uint32_t yh = __builtin_amdgcn_ubfe(q0, ph, 1);
                            if (NP > 1) yh |= __builtin_amdgcn_ubfe(q1, ph, 1) << 1;
                            if (NP > 2) yh |= __builtin_amdgcn_ubfe(q2, ph, 1) << 2;
                            const uint32_t hq = left ? 1u << (8u + yh) : 0u;
                            const uint32_t r2 = ((qr + (T0 & 0xFFFF0000u)) & 0xFFFF0000u) | (qr & 0xFFu & ~(1u << ys)) | (again ? 1u << ys : 0u) | hq;
                            worst = max(worst, (int)r2 >> 16);
                            lds_store(rq + NP * kRow, left);
                            lds_store(rq + (NP + 1) * kRow, r2);
                            const uint32_t ob = 1u << dd, sm = lds_load(G.smask + (dd << 2));
                            RD = r2 & 0xFFu ? RD | ob : RD & ~ob;
                            HD = r2 & (r2 >> 8) & sm ? HD | ob : HD & ~ob;
                            head_moved(dd << NP, qr >> 8 & 0xFFu, hq >> 8);
                        }
                    }
                }
                entry = (T0 & 63u) | (w >> mushift) << 6;
                // the consumers: one more micro-batch waits.  (No consumer: the row that
                // stays zero, increment 0, and the block's own record.)
                uint32_t dc_before = 0, now_before = 0;
                for (int k = 0;;) {
                    const uint32_t wc2 = wc + C1;
                    const bool runs_now = ready(wc2);
                    const uint32_t dc = (C0 >> 3) & 31u, bit = 1u << (C0 & 7u);
                    lds_store(cwa, wc2);
                    if (TP) {
                        const uint32_t cg = ((C0 & 0xFF00u) - G.wrow) / kRow;        // (the zero row lies behind the types')
                        const uint32_t cm = cg < (uint32_t)K ? lds_load(G.tpm + cg * 4u) : 0u;
                        if (runs_now) {
                            if (cm) {
                                const uint32_t i = (lds_load(G.tpi + cg * 4u) & 63u) / 6u;
                                rtp |= 1u << i;
                                RD |= cm;
                                for (uint32_t rest_d = cm; rest_d; rest_d &= rest_d - 1u) {
                                    const uint32_t dd = (uint32_t)__builtin_ctz(rest_d), rq = dd * RS + rec0 + (NP + 1) * kRow;
                                    lds_store(rq, lds_load(rq) | 1u << lds_load(G.tps + (i * 32u + dd) * 4u));
                                }
                            } else {
                                const uint32_t now = lds_load(cra) | bit;
                                lds_store(cra, now);
                                RD |= 1u << dc;
                                HD |= now & (now >> 8) & lds_load(G.smask + (dc << 2)) ? 1u << dc : 0u;
                            }
                        }
                    } else {
                        uint32_t now = k == 0 ? (dc == d ? rhm2 : rc) : k == 1 ? (dc == dc_before ? now_before : dc == d ? rhm2 : rc) : lds_load(cra);
                        now |= runs_now ? bit : 0u;
                        lds_store(cra, now);
                        RD |= (now & 0xFFu ? 1u : 0u) << dc;
                        HD |= (now & (now >> 8) & 0xFFu ? 1u : 0u) << dc;
                        dc_before = dc; now_before = now;
                    }
                    if (CHAIN || ++k >= maxout) break;
                    if (KIND == 1 && k == 1) {
                        C0 = E0; C1 = E1; wc = wd; rc = rd;
                        cwa = (C0 & 0xFF00u) + lane4; cra = (C0 >> 16) + lane4;
                        continue;
                    }
                    lds_load2(ca + 8u + 8u * (uint32_t)k, C0, C1);
                    cwa = (C0 & 0xFF00u) + lane4; cra = (C0 >> 16) + lane4;
                    wc = lds_load(cwa);
                }
            }
            return entry;
        };
        const int full = total / 2;
        whole = any;
        for (int wi = 0; any && wi < full; wi++) {
            const uint32_t e0 = step(), e1 = step();
            prog[(size_t)wi * kProgRow] = e0 | e1 << 16;
            if (!REPAIR || (wi & 7) == 7) {
                if (__builtin_expect((wi & 7) == 7 && turns != 0, 0)) take_turn(turns);
                const bool going = valid && (REPAIR ? !(drop_mem && worst > M) : building);
                if (__ballot(going) == 0) { whole = false; break; }
            }
        }
        if (whole && (total & 1)) prog[(size_t)full * kProgRow] = step();
        }
        // ---- verdict
        int peak = worst;
        if (status == kOk) {
            if (idle) peak = max(peak, 0);                       // a device without blocks holds nothing
            if (peak > M) status = kMem;
        }
        const bool rejected = valid && status != kOk, ok = valid && status == kOk;
        nev += (uint32_t)__builtin_popcountll(__ballot(rejected));
#pragma unroll
        for (int s = 1; s < kNumStatus; s++) cnt[s] += (uint32_t)__builtin_popcountll(__ballot(rejected && status == s));
        if (rejected) {
            if (code_out) code_out[idx - first] = -status;
            if (peak_out) peak_out[idx - first] = status == kMem ? peak : 0;
        }
        if (ok) {
            uint32_t *meta = slots + slot;
            meta[0] = (uint32_t)idx; meta[kProgRow] = (uint32_t)(idx >> 32); meta[2 * kProgRow] = (uint32_t)peak;
            // (all N_R occurrences are placed: next micro-batch - N_R is the lead)
            for (int r = 0; r < P.ntok; r += 4) {
                uint32_t pack = 0;
                for (int q = 0; q < 4 && r + q < P.ntok; q++) {
                    const uint32_t h = G.head[r + q], w = lds_load((h & 0xFFFFu) + lane4);
                    pack |= (CODES ? __builtin_amdgcn_ubfe(w, h >> 16 & 31u, h >> 24) : (w >> mushift) - NR) << (8 * q);
                }
                meta[(size_t)(3 + r / 4) * kProgRow] = pack;
            }
            lds_store8(st_row + slot, 1u);
        }
    };

    // ---------------------------------------------------------------- window sweeps of up to 64 candidates in state `cls`
    // Times, rings and boundary as in the general kernel; eigenvector test after every sweep.
    auto sweep = [&](uint32_t cls, bool more_to_come) {
        uint32_t slot = 0;
        lds_store8(sel_row + (uint32_t)lane, (uint32_t)lane);
        __syncthreads();
        const uint32_t n = slots_in(cls, true, slot);
        const bool have = (uint32_t)lane < n;
        // (a lane without a candidate runs the first one's program and drops the result)
        if (CODES && !have) slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
        const uint32_t *meta = slots + slot, *prog = progs + slot;
        __threadfence_block();                                   // the wave's other lanes wrote these words
        const uint64_t idx = have ? (uint64_t)meta[0] | ((uint64_t)meta[kProgRow] << 32) : first;
        const int pk = (int)meta[2 * kProgRow];
        const uint32_t st0 = G.state + lane_s, prev0 = G.prev + lane_s;
        for (int r = 0; r < P.ntok; r += 4) lds_store(G.leads + (uint32_t)(r / 4) * kRow + lane4, have ? meta[(size_t)(3 + r / 4) * kProgRow] : 0u);
        for (int s = 0; s < P.nslots; s++) time_store(st0 + (uint32_t)s * SROW, 0u);
        for (int d = 0; d < D + G.apart_rows; d++) time_store(prev0 + (uint32_t)d * SROW, 0u);       // (and what lies behind these)
        const int maxin = G.maxin;
        auto block = [&](uint32_t e, uint32_t A, uint32_t B, uint32_t pr) {
            const uint32_t mu8 = (e >> 6) * SROW, da = (B & 0xFFFFu) + lane_s;
            if (CHAIN) {
                const uint32_t ta = (B >> 16) + mu8 + lane_s;
                const uint32_t en = max(time_load(da), time_load(ta)) + (A & 0xFFFFFFu);
                time_store(da, en);
                time_store(ta, en);
                return;
            }
            const uint32_t g4 = (e & 63u) << 2;
            uint32_t s = 0;
            const uint32_t mask = TP ? lds_load(G.tpm + g4) : 0u;
            s = lds_load(da);
            for (uint32_t rest = mask; rest; rest &= rest - 1u) s = max(s, lds_load(st0 + (uint32_t)__builtin_ctz(rest) * kRow));
            for (int k = 0;;) {
                s = max(s, max(lds_load((pr & 0xFFFFu) + mu8 + lane4), lds_load((pr >> 16) + mu8 + lane4)));
                if ((k += 2) >= maxin) break;
                pr = lds_load(G.swp + (uint32_t)k / 2u * (uint32_t)K * 4u + g4);
            }
            const uint32_t en = s + (A & 0xFFFFFFu);
            lds_store(da, en);
            for (uint32_t rest = mask; rest; rest &= rest - 1u) lds_store(st0 + (uint32_t)__builtin_ctz(rest) * kRow, en);
            lds_store((B >> 16) + (mu8 & (uint32_t)((int)A >> 31)) + lane4, en);
        };
        // Eight blocks of a chain problem's program.  A block's two times are read before the block before has written its own,
        // which it takes from a register where they share the device or the ring entry (end times only grow, so the largest of the
        // three is right): the reads' latency, two thirds of a block's time at one to three waves a SIMD, overlaps.
        auto codes_word = [&](const uint32_t (&cur)[4], int left) {
            // (GraphTab::sw)
            constexpr uint32_t table = GRAPH ? 8u * 128u : W64 ? 6u * 256u : (NP <= 1 ? 4u : 5u) * 128u;
            uint32_t da[8], ta[8], t[8], pa[8], pb[8];           // (graphs: ta is written only, and the two producers' entries are read)
            auto look_up = [&](bool all) {
                uint32_t e[8], B[8], from[8];
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    // (a word past the last block was never written: its type is taken as 0, and nothing of it is used)
                    e[q] = !all && q >= left ? 0u : q & 1 ? cur[q / 2] >> 16 : cur[q / 2] & 0xFFFFu;
                    const uint32_t at = GRAPH ? ((e[q] & 0x1F8u) << 1) + table : (e[q] & 0x1F8u) + table;
                    lds_load2(at, t[q], B[q]);
                    from[q] = GRAPH ? lds_load(at + 8u) : 0u;
                }
                __builtin_amdgcn_sched_barrier(0);               // (all eight on their way before the first is waited for)
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    da[q] = (B[q] & 0xFFFFu) + lane_s;
                    const uint32_t mu = (e[q] >> 2 & 0xF80u) | lane_s;
                    ta[q] = (B[q] >> 16) + mu;
                    pa[q] = GRAPH ? (from[q] & 0xFFFFu) + mu : ta[q];
                    pb[q] = GRAPH ? (from[q] >> 16) + mu : 0u;
                }
            };
            uint32_t fr, tk, tk_b = 0, before = 0;
            auto one = [&](int q, bool more) {
                uint32_t fr2 = 0, tk2 = 0, tk_b2 = 0;
                if (more) { fr2 = time_load(da[q + 1]); tk2 = time_load(pa[q + 1]); if (GRAPH) tk_b2 = time_load(pb[q + 1]); }
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t wrote = ta[q - (q > 0)];
                const bool shared = q > 0 && (da[q] == da[q - (q > 0)] || pa[q] == wrote || (GRAPH && pb[q] == wrote));
                const uint32_t en = max(max(GRAPH ? max(fr, tk_b) : fr, tk), shared ? before : 0u) + t[q];
                time_store(da[q], en);
                time_store(ta[q], en);
                __builtin_amdgcn_sched_barrier(0);
                before = en; fr = fr2; tk = tk2; tk_b = tk_b2;
            };
            if (left >= 8) {
                look_up(true);
                fr = time_load(da[0]); tk = time_load(pa[0]); if (GRAPH) tk_b = time_load(pb[0]);
#pragma unroll
                for (int q = 0; q < 8; q++) one(q, q < 7);
            } else {
                look_up(false);
                fr = time_load(da[0]); tk = time_load(pa[0]); if (GRAPH) tk_b = time_load(pb[0]);
#pragma unroll
                for (int q = 0; q < 7; q++) if (q < left) one(q, q + 1 < left);
            }
        };
        uint32_t T = 0;
        bool done = !have;
        const int tries = cls == 1u ? G.first_tries : G.retry_tries;
        const bool settle = cls != 1u && D + P.ntok * (int)NR <= 128;        // (one bit per value)
        uint32_t top_before = 0;
        uint64_t was_lo = 0, was_hi = 0;
        for (int j = 0;; j++) {
            const uint32_t open = (uint32_t)__builtin_popcountll(__ballot(!done));
            if (open == 0) break;
            // The first pass goes on while many lanes are open; a few stragglers wait until 64 of them fill a wave.  (One
            // more sweep here costs the wave one sweep; a straggler costs a restart of three or more sweeps of 64 lanes.)
            if (cls == 1u ? j >= tries && (tries == 0 || j >= 8 || (open <= 20u && more_to_come)) : j >= tries) break;
            // four program words (eight blocks) at a time, the next four on their way
            uint32_t cur[4], nxt[4];
#pragma unroll
            for (int q = 0; q < 4; q++) cur[q] = prog[(size_t)q * kProgRow];
            for (int wi = 0; wi < nwords; wi += 4) {
                if (__builtin_expect((wi & 12) == 0 && turns != 0, 0)) take_turn(turns);
                const int ahead = wi + 4 < nwords ? wi + 4 : wi;
#pragma unroll
                for (int q = 0; q < 4; q++) nxt[q] = prog[(size_t)(ahead + q) * kProgRow];
                const int left = total - 2 * wi;                 // blocks from here on
                if constexpr (CODES) {
                    codes_word(cur, left);
#pragma unroll
                    for (int q = 0; q < 4; q++) cur[q] = nxt[q];
                    continue;
                }
                uint32_t e[8], A[8], B[8], pr[8];
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    // (a word past the last block was never written, and a lane without a candidate has stale ones: type and
                    // micro-batch stay inside the tables and the rings, or are not used)
                    e[q] = q & 1 ? cur[q / 2] >> 16 : cur[q / 2] & 0xFFFFu;
                    if (!have) e[q] = 0;
                    const uint32_t g4 = (e[q] & 63u) << 2;
                    lds_load2(G.sw + 2u * g4, A[q], B[q]);
                    pr[q] = !CHAIN ? lds_load(G.swp + g4) : 0u;
                }
#pragma unroll
                for (int q = 0; q < 8; q++) if (q < left) block(e[q], A[q], B[q], pr[q]);
#pragma unroll
                for (int q = 0; q < 4; q++) cur[q] = nxt[q];
            }
            // Window boundary: micro-batches mu >= N_R are mu - N_R of the next window.  Every value that crosses it and
            // means anything (devices with blocks, ring entries below the lead of the ring's first type) grew by the same
            // amount: an eigenvector, and the amount is the period.  In the longer search also: the largest growth D was
            // that of the boundary before, and every value that grew by D then grew by D now.  No cycle ratio exceeds the
            // largest growth; and a value that grew by D got its time from one that grew by D the time before (that
            // one's growth bounds its own from above), which is again one of these, so following them closes a cycle
            // of ratio D.  (Forward-only pipelines need this: devices before the slowest keep a smaller growth for ever.)
            // (Values by fours: their loads are on their way together.  One by one, with the loads' latency and the bookkeeping in
            // lane masks, a boundary cost 40 to 60 % of the sweeps of graphs with many short rings.)
            // From the seventh sweep of the longer search on, two windows at a time: the same two tests on the map of two windows, whose ratio
            // is twice the period's.  (A cycle through two windows whose time is odd makes the values grow by turns. One candidate in 4,000 of
            // the diamond at three micro-batches; all others settle within four sweeps. On its way through the general kernel's
            // list that one cost a call of 100,003 candidates 360 of 421 us.)
            const bool two = settle && G.apart && j >= kTwoWindows;
            if (two && ((j - kTwoWindows) & 1) == 0) {
                for (int r = 0; r < P.ntok; r++) {
                    const uint32_t base = st0 + (G.ring[r] & 0xFFFFu) * SROW, lg = (lds_load(G.leads + (uint32_t)(r / 4) * kRow + lane4) >> (8 * (r & 3))) & 255u;
                    for (uint32_t m = 0; m < NR; m++) {
                        const uint32_t x = time_load(base + (m + NR) * SROW);
                        time_store(base + m * SROW, m < lg ? x : 0u);
                        time_store(base + (m + NR) * SROW, 0u);
                    }
                }
                if (j == kTwoWindows) top_before = ~0u;
                continue;
            }
            auto in_flight = [&](int r) -> uint32_t {
                return (lds_load(G.leads + (uint32_t)(r / 4) * kRow + lane4) >> (8 * (r & 3))) & 255u;
            };
            auto values = [&](auto &&device, auto &&ring) {
                for (int d = 0; d < D; d += 4) {
                    uint32_t x[4], old[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) {                // (past the last one: the last one again)
                        const uint32_t at = (uint32_t)min(d + q, D - 1) * SROW;
                        x[q] = time_load(st0 + at); old[q] = time_load(prev0 + at);
                    }
#pragma unroll
                    for (int q = 0; q < 4; q++) device(min(d + q, D - 1), x[q], x[q] - old[q]);
                }
                if (NR <= 2u) {
                    // (few values a ring: two rings at a time.  Fours of one ring, the same value up to four times, cost graphs of one
                    // micro-batch a window 12 % of the kernel.)
                    for (int r = 0; r < P.ntok; r += 2)
                        for (uint32_t m = 0; m < NR; m++) {
                            uint32_t x[2], old[2], base[2], kept[2];
#pragma unroll
                            for (int q = 0; q < 2; q++) {
                                const uint32_t rows = G.ring[min(r + q, P.ntok - 1)];
                                base[q] = st0 + ((rows & 0xFFFFu) + m) * SROW; kept[q] = st0 + ((rows >> 16) + m) * SROW;
                                x[q] = time_load(base[q] + NR * SROW); old[q] = time_load(kept[q]);
                            }
#pragma unroll
                            for (int q = 0; q < 2; q++) {
                                const int rq = min(r + q, P.ntok - 1);
                                ring(base[q], kept[q], (uint32_t)D + (uint32_t)rq * NR + m, m < in_flight(rq), x[q], x[q] - old[q]);
                            }
                        }
                    return;
                }
                for (int r = 0; r < P.ntok; r++) {
                    const uint32_t rows = G.ring[r], base = st0 + (rows & 0xFFFFu) * SROW, kept = st0 + (rows >> 16) * SROW, lg = in_flight(r);
                    for (uint32_t m = 0; m < NR; m += 4) {
                        uint32_t x[4], old[4];
#pragma unroll
                        for (uint32_t q = 0; q < 4; q++) {
                            const uint32_t at = min(m + q, NR - 1u) * SROW;
                            x[q] = time_load(base + at + NR * SROW); old[q] = time_load(kept + at);
                        }
#pragma unroll
                        for (uint32_t q = 0; q < 4; q++) {
                            const uint32_t n = min(m + q, NR - 1u);
                            ring(base + n * SROW, kept + n * SROW, (uint32_t)D + (uint32_t)r * NR + n, n < lg, x[q], x[q] - old[q]);
                        }
                    }
                }
            };
            uint32_t least = 0xFFFFFFFFu, top = 0;               // growths
            auto grew = [&](uint32_t by, bool on) { least = min(least, on ? by : 0xFFFFFFFFu); top = max(top, on ? by : 0u); };
            if (settle)
                values([&](int d, uint32_t, uint32_t by) { grew(by, (busy >> d & 1u) != 0); },
                       [&](uint32_t, uint32_t, uint32_t, bool on, uint32_t, uint32_t by) { grew(by, on); });
            uint64_t now_lo = 0, now_hi = 0;                     // the values that grew by that much, a bit each
            auto note = [&](uint32_t v, uint32_t by, bool on) {
                if (!settle) { grew(by, on); return; }
                if (v < 64u) now_lo |= on && by == top ? 1ull << v : 0ull; else now_hi |= on && by == top ? 1ull << (v & 63u) : 0ull;
            };
            values([&](int d, uint32_t x, uint32_t by) {
                       time_store(prev0 + (uint32_t)d * SROW, x);
                       note((uint32_t)d, by, (busy >> d & 1u) != 0);
                   },
                   [&](uint32_t base, uint32_t kept, uint32_t v, bool on, uint32_t x, uint32_t by) {
                       note(v, by, on);
                       const uint32_t keep = on ? x : 0u;
                       time_store(base, keep);
                       time_store(kept, keep);
                       time_store(base + NR * SROW, 0u);
                   });
            if (settle) {
                const bool held = j > 0 && top == top_before && (was_lo & ~now_lo) == 0 && (was_hi & ~now_hi) == 0;
                if (!done && held) { T = two ? (top + 1u) / 2u : top; done = true; }
                top_before = top; was_lo = now_lo; was_hi = now_hi;
            }
            if (!done && least == top) { T = two ? (top + 1u) / 2u : top; done = true; }
        }
        const bool scored = have && done, left_open = have && !done;
        const uint32_t ns = (uint32_t)__builtin_popcountll(__ballot(scored));
        nev += ns;
        cnt[kOk] += ns;
        if (scored) {
            if (key_less((int)T, idx, best, best_idx)) { best = (int)T; best_idx = idx; }
            if (code_out) code_out[idx - first] = (int)T;
            if (peak_out) peak_out[idx - first] = pk;
        }
        if (left_open && cls != 1u) {
            const uint32_t at = atomicAdd(out_count, 1u);
            if (at < out_cap) out_list[at] = idx;                // (more than that: the general kernel scores the whole range)
        }
        if (cls == 1u) nretry += (uint32_t)__builtin_popcountll(__ballot(left_open));
        if (have) lds_store8(st_row + slot, left_open && cls == 1u ? 2u : 0u);
        __syncthreads();
    };

    const uint64_t stride = (uint64_t)gridDim.x * kWave;
    const uint64_t rounds = (count + stride - 1) / stride;          // the same trip count for every lane of the grid
    for (uint64_t r = 0;;) {
        uint32_t unused;
        const uint32_t n1 = slots_in(1u, false, unused), n2 = slots_in(2u, false, unused);
        // (a wave whose share has ended early does no more rounds)
        const bool fresh = r < rounds && r * stride + (uint64_t)blockIdx.x * kWave < count;
        if (!fresh && n1 > 0 && n1 + n2 <= (uint32_t)kWave) {
            // the last candidates of the share, stragglers among them: one longer search for all
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const uint32_t a = st_row + (uint32_t)(j * kWave + lane);
                if (lds_load8(a) == 1u) lds_store8(a, 2u);
            }
            __syncthreads();
            sweep(2u, true);
        } else if (n2 >= (uint32_t)kWave || (!fresh && n1 == 0 && n2 > 0)) sweep(2u, true);
        else if (n1 >= (uint32_t)kWave || (!fresh && n1 > 0)) sweep(1u, fresh || n1 > (uint32_t)kWave || n2 > 0);
        else if (fresh) {
            const uint64_t kk = r++ * stride + (uint64_t)blockIdx.x * kWave + lane;
            const bool valid = kk < count;
            build(valid ? first + kk : first, valid);
            __syncthreads();
            if (r == 1 && slots_in(1u, false, unused) >= 7u * (uint32_t)kWave / 8u) {
                turns = in_last ? waves.last : waves.others;
                __builtin_amdgcn_s_setprio(0);
            }
        } else break;
    }
    if (!recs) return;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        int op = __shfl_xor(best, off);
        uint32_t ilo = __shfl_xor((uint32_t)best_idx, off), ihi = __shfl_xor((uint32_t)(best_idx >> 32), off);
        uint64_t oi = ((uint64_t)ihi << 32) | ilo;
        if (key_less(op, oi, best, best_idx)) { best = op; best_idx = oi; }
    }
    if (lane == 0) {
        BlockRec rr;
        // (window sweeps and blocks placed are reported for the fast kernel only)
        rr.period = best; rr.n_retried = nretry; rr.index = best_idx; rr.n_evaluated = nev; rr.n_sweeps = 0; rr.n_blocks = 0; rr.n_high = 0;
#pragma unroll
        for (int s = 0; s < kNumStatus; s++) rr.n_status[s] = cnt[s];
        recs[blockIdx.x] = rr;
    }
}

// ------------------------------------------------------------------ launcher
typedef void (*graph_fn)(const KParams *, const GraphTab *, uint64_t, uint64_t, BlockRec *, int32_t *, int32_t *, uint64_t *, uint32_t *,
                         uint32_t, uint32_t *, uint32_t *, GraphTurns);

template <bool REPAIR, int KIND>
static graph_fn pick_np(int np)
{
    if constexpr (KIND >= 3) if (np == 0) return eval_graph_kernel<0, REPAIR, KIND>;
    return np == 1 ? eval_graph_kernel<1, REPAIR, KIND> : np == 2 ? eval_graph_kernel<2, REPAIR, KIND> : eval_graph_kernel<3, REPAIR, KIND>;
}

template <bool REPAIR>
static graph_fn pick_kind(const KParams &kp)
{
    if (kp.tp) return pick_np<REPAIR, 2>(kp.graph_np);
    if (kp.graph_codes == 3) return eval_graph_kernel<0, REPAIR, 5>;
    if (kp.graph_codes) return kp.graph_codes == 1 ? pick_np<REPAIR, 3>(kp.graph_np) : pick_np<REPAIR, 4>(kp.graph_np);
    return kp.graph_chain ? pick_np<REPAIR, 0>(kp.graph_np) : pick_np<REPAIR, 1>(kp.graph_np);
}

static graph_fn pick_graph(const KParams &kp) { return kp.space == kSampledRepair ? pick_kind<true>(kp) : pick_kind<false>(kp); }

const void *graph_kernel(const KParams &kp) { return (const void *)pick_graph(kp); }

int launch_graph(const KParams &kp, uint64_t first, uint64_t count, int blocks, void *recs, int32_t *code, int32_t *peak, void *ws,
                 uint32_t *slots, GraphTurns turns, void *stream)
{
    DevResult *res = (DevResult *)((char *)ws + kWsResultOff);
    hipLaunchKernelGGL(pick_graph(kp), dim3(blocks), dim3(kWave), kp.graph_lds, (hipStream_t)stream, (const KParams *)((char *)ws + kWsParamsOff),
                       (const GraphTab *)((char *)ws + kp.graph_at), first, count, (BlockRec *)recs, code, peak,
                       (uint64_t *)((char *)ws + kWsListOff), &res->defer_count, kWsListCap, &res->overflow, slots, turns);
    return (int)hipGetLastError();
}

}  // namespace tessel
