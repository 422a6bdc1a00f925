// Host side of the C ABI declared in include/tessel.h: validation of the problem statement
// (Sec. III-A of the Tessel paper), static tables for the kernels, launches, result read-back,
// and schedule completion (Sec. IV-C) for the best repetend.  All candidate scoring is done
// by the kernels in tessel_kernels.hip; nothing here falls back to the CPU for it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cstdlib>
#include <cstdint>
#include <cstring>
#include <atomic>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "../../include/tessel.h"
#include "tessel_device.h"

using namespace tessel;

namespace tessel { size_t block_rec_bytes(int blocks); }

struct tessel_problem {
    uint64_t id = 0;                    // never reused: names the handle as the owner of a workspace
    KParams kp;
    GraphTab graph;                     // tables of the graph kernel (graph.ok)
    std::vector<int32_t> t, m;
    std::vector<uint32_t> mask;
    std::vector<int32_t> dep_src, dep_dst;
    std::vector<int8_t> leadtab;        // CANONICAL
    std::vector<uint64_t> wtab;         // CANONICAL
    // What a workspace starts with, copied in one piece: an empty record, the parameters, and from kWsTablesOff on (CANONICAL) the two
    // tables, where they are small KParams::orders and leadrows, and the graph kernel's tables, each from a multiple of 256 bytes on
    std::vector<char> image;
    size_t table_at[4] = {0, 0, 0, 0};
    uint64_t nlead = 0;
    uint64_t count = 0;
    int num_cus = 0;
    void *ws = nullptr;                 // workspace the running best lives in
    int max_blocks = 0;                 // 0, or the largest grid that workspace has queues for (the library's own buffer)
    bool ws_ready = false;
    hipStream_t stream = nullptr;
    int last_hip = 0;
    bool force_general = false;         // TESSEL_FORCE_GENERAL=1: score with the general kernel only
    bool mail = true;                   // TESSEL_MAIL=0 (test knob): results are copied, as where no box is free
    Detail detail;
    DevResult result;
    std::vector<int32_t> starts;        // least start times of the decoded candidate, by type * N_R + occurrence
    bool period_right = false;          // ... and whether the record's period is its least one
    // index ranges scored since the last reset (adjacent ones merged), and whether launches are cut into the
    // small pieces in which no list of unfinished candidates can overflow
    std::vector<std::pair<uint64_t, uint64_t>> ranges;
    bool safe_pieces = false;
    bool best_dirty = true;             // candidates were scored (or the search was reset) since the best was fetched
    // searched completion
    bool comp_ready = false;            // CompParams of (comp_index, N, J) are in the workspace
    uint64_t comp_index = 0;            // best candidate they were built for
    CompParams comp;
    CompMatrix comp_matrix;
};

static_assert(kScratchBytes == TESSEL_NOALLOC_SCRATCH_BYTES, "header and library disagree on the size of the library's own workspace");

static int hip_fail(tessel_problem *p, int e) { p->last_hip = e; return TESSEL_E_HIP; }

// Which handle a device workspace belongs to.  The kernels read the problem's parameter block, the running best and
// the queues from the workspace itself, so a buffer serves one handle at a time: binding it to another handle ends
// the first one's search, and that handle's next scoring call binds it anew (a new search), while its calls that
// read results are refused.  (Host memory only; the one piece of state shared between handles.)
namespace {
std::mutex g_owner_mutex;
std::unordered_map<const void *, uint64_t> g_owner;
std::atomic<uint64_t> g_next_id{1};

bool owns_workspace(const tessel_problem *p)
{
    if (!p->ws || !p->ws_ready) return false;
    std::lock_guard<std::mutex> lock(g_owner_mutex);
    auto it = g_owner.find(p->ws);
    return it != g_owner.end() && it->second == p->id;
}
void take_workspace(const tessel_problem *p, const void *ws)
{
    std::lock_guard<std::mutex> lock(g_owner_mutex);
    g_owner[ws] = p->id;
}
void release_workspaces(const tessel_problem *p)
{
    std::lock_guard<std::mutex> lock(g_owner_mutex);
    for (auto it = g_owner.begin(); it != g_owner.end();)
        if (it->second == p->id) it = g_owner.erase(it); else ++it;
}
}  // namespace

extern "C" const char *tessel_strerror(int code)
{
    switch (code) {
    case TESSEL_OK: return "ok";
    case TESSEL_E_INVALID_ARG: return "invalid argument";
    case TESSEL_E_BAD_DEP: return "dependency graph of a micro-batch has a cycle";
    case TESSEL_E_UNBALANCED_MEMORY: return "memory deltas on a device do not sum to zero";
    case TESSEL_E_TOOBIG: return "count or time bound too large";
    case TESSEL_E_WORKSPACE: return "workspace missing, misaligned or too small, or a launch overflowed its retry list (submit smaller ranges)";
    case TESSEL_E_HIP: return "HIP runtime error";
    case TESSEL_E_NO_FEASIBLE: return "no feasible candidate scored";
    case TESSEL_E_RANGE: return "range outside the candidate space or too few micro-batches";
    case TESSEL_E_UNSUPPORTED: return "problem outside the limits of this implementation";
    case TESSEL_E_NO_SCHEDULE: return "no warm-up/cool-down order fits the memory cap";
    default: return "unknown error";
    }
}

// number of distinct sequences of a multiset; 0 on 64-bit overflow
static uint64_t multiset_sequences(const int *cnt, int ntypes)
{
    unsigned __int128 r = 1;
    unsigned placed = 0;
    for (int y = 0; y < ntypes; y++)
        for (int k = 1; k <= cnt[y]; k++) {
            placed++;
            r = r * placed / (unsigned)k;
            if (r >> 64) return 0;
        }
    return (uint64_t)r;
}

// lead vectors of the CANONICAL space: Property 2 on every dependency, minimum 0,
// lexicographic with type 0 most significant
static bool gen_leads(const tessel_problem &p, int K, int NR, std::vector<int8_t> &tab, size_t limit)
{
    std::vector<int> cur(K, 0);
    int i = 0;
    cur[0] = -1;
    while (i >= 0) {
        cur[i]++;
        if (cur[i] >= NR) { i--; continue; }
        bool ok = true;
        for (size_t e = 0; e < p.dep_src.size() && ok; e++) {
            int a = p.dep_src[e], b = p.dep_dst[e];
            if (std::max(a, b) == i && cur[a] < cur[b]) ok = false;
        }
        if (!ok) continue;
        if (i == K - 1) {
            if (*std::min_element(cur.begin(), cur.end()) == 0) {
                if (tab.size() / K >= limit) return false;
                for (int k = 0; k < K; k++) tab.push_back((int8_t)cur[k]);
            }
        } else {
            i++;
            cur[i] = -1;
        }
    }
    return true;
}

// The same for chains on masks by code (GraphTab::codes); false: not such a problem, or a field of its records would not
// hold it (memory prefixes, times of a window sweep in 16 bits; a dependency listed twice draws twice).
static bool code_tables(const tessel_problem &p, GraphTab &gt, const std::vector<std::vector<int>> &in, const std::vector<std::vector<int>> &outs,
                        long span_max)
{
    const KParams &kp = p.kp;
    const int D = kp.D, K = kp.K, NR = kp.NR, nb = gt.np;
    if (!gt.chain || kp.tp || (D << nb) > 64 || (kp.space != kSampledStrict && kp.space != kSampledRepair)) return false;
    size_t distinct = 0;
    for (int i = 0; i < K; i++) distinct += in[i].size();
    if (distinct != p.dep_src.size()) return false;
    if (span_max > (nb == 1 ? 8000 : nb == 2 ? 30000 : 120)) return false;
    // end times of the last sweep of all: at most the serial time of the windows so far
    if ((int64_t)kp.UB * (std::max(9, gt.retry_tries) + 1) > 65535) return false;
    const bool packed = nb == 1 && NR <= 8;
    const uint32_t row = kWave * 4, half = row / 2, ts = (D << nb) > 32 ? 256 : 128;
    const int rows = packed ? 2 : nb == 1 ? 3 : nb + 3, row_w = packed ? 1 : nb + 1, row_l = nb == 1 ? row_w : nb + 2;
    const int words = ts == 256 ? 6 : nb == 1 ? 4 : 5;
    uint32_t at = (uint32_t)words * ts;
    gt.sw = at; at += (uint32_t)K * 8;
    gt.ntab = (int)(at / 4);
    at = (at + row - 1) / row * row;
    gt.slot_rows = at; at += row;
    gt.rec = at;
    const uint32_t build_end = at + (uint32_t)(D * rows) * row;
    gt.state = at; at += (uint32_t)kp.nslots * half;
    gt.prev = at; at += (uint32_t)D * half;
    gt.strash = at; at += half;
    at = (at + row - 1) / row * row;
    gt.leads = at; at += (uint32_t)((kp.ntok + 3) / 4) * row;
    gt.lds_bytes = std::max(build_end, at);
    memset(gt.tab, 0, sizeof gt.tab);
    gt.codes = ts == 256 ? 2 : 1;
    gt.apart = 1;                                            // (a chain's types share its ring: KParams::ring_kept)
    gt.np = packed ? 0 : nb;
    std::vector<int> code(K, 0);
    for (int d = 0; d < D; d++)
        for (int y = 0; y < kp.ntd[d]; y++)
            code[(y < 4 ? kp.type_of[d] >> (8 * y) : kp.type_of_hi[d] >> (8 * (y - 4))) & 0xFFu] = (d << nb) + y;
    auto dev = [&](int g) -> int { return code[g] >> nb; };
    auto sym = [&](int g) -> int { return code[g] & ((1 << nb) - 1); };
    auto wait_at = [&](int g) -> int { return nb == 3 ? 4 * sym(g) : 5 * sym(g); };
    auto lead_at = [&](int g) -> int { return nb == 1 ? 10 + 4 * sym(g) : nb == 2 ? 4 * sym(g) : 3 * sym(g); };
    const int mem_at = nb == 1 ? 18 : nb == 2 ? 16 : 24;
    auto word = [&](int w, int c) -> uint32_t & { return gt.tab[((uint32_t)w * ts) / 4 + (uint32_t)c]; };
    auto rec_row = [&](int d, int r) -> uint32_t { return gt.rec + (uint32_t)(d * rows + r) * row; };
    for (int g = 0; g < K; g++) {
        const int c = code[g], h = outs[g].empty() ? -1 : outs[g][0];
        const bool same = h >= 0 && dev(h) == dev(g);
        const uint32_t mem = (uint32_t)p.m[g] << mem_at, inc = h >= 0 ? 1u << wait_at(h) : 0u;
        word(0, c) = (nb == 1 ? mem : 0u) - (1u << wait_at(g)) + (same ? inc : 0u);
        word(1, c) = h >= 0 && code[h] < 32 ? 1u << code[h] : 0u;
        word(2, c) = rec_row(h >= 0 && !same ? dev(h) : dev(g), row_w) | ((uint32_t)g * 8u + ((uint32_t)(NR - 1) << 9)) << 16;
        word(3, c) = same ? 0u : inc;
        if (words > 4) word(4, c) = mem;
        if (words > 5) word(5, c) = h >= 0 && code[h] >= 32 ? 1u << (code[h] - 32) : 0u;
        auto ring_address = [&](int i) -> uint32_t { return gt.state + (uint32_t)kp.tokbase[i] * half; };
        gt.tab[gt.sw / 4 + 2 * g] = (uint32_t)p.t[g];
        gt.tab[gt.sw / 4 + 2 * g + 1] = (gt.state + (uint32_t)dev(g) * half) | ring_address(kp.tokbase[g] != kNoRing ? g : in[g][0]) << 16;
    }
    int n = 0;
    for (int last = 0; last < K; last++) {
        if (!outs[last].empty()) continue;
        for (int g = last;; g = in[g][0]) {
            uint32_t *e = gt.links[n++];
            uint32_t number = 0, cross = 0;
            for (int k = 0; k < kp.ndeps; k++) if (kp.dsrc[k] == g) { number = (uint32_t)k; cross = kp.dcross[k] != 0; }
            e[0] = rec_row(dev(g), row_w) | number << 16 | cross << 24 | (uint32_t)outs[g].empty() << 25 | (uint32_t)in[g].empty() << 26;
            e[1] = (uint32_t)wait_at(g) | (uint32_t)code[g] << 8 | (uint32_t)lead_at(g) << 16;
            e[2] = (uint32_t)kp.fixed[g] << 28;
            e[3] = (uint32_t)p.m[g] << mem_at;
            if (in[g].empty()) break;
        }
    }
    for (int r = 0; r < kp.ntok; r++) {
        const int g = kp.ring_head[r];
        gt.head[r] = rec_row(dev(g), row_l) | (uint32_t)lead_at(g) << 16 | (nb == 3 ? 3u : 4u) << 24;
    }
    gt.ok = 1;
    return true;
}

// The same for graphs with up to two producers and two consumers a type, on single devices with up to two types, 32 codes, windows of 8
// micro-batches and 16 types (a lead is four bits of one register pair).
static bool graph_code_tables(const tessel_problem &p, GraphTab &gt, const std::vector<std::vector<int>> &in, const std::vector<std::vector<int>> &outs,
                              long span_max)
{
    const KParams &kp = p.kp;
    const int D = kp.D, K = kp.K, NR = kp.NR;
    constexpr int most_types = 16, most_nr = 8, most_devices = 16;
    if (gt.chain || kp.tp || gt.np != 1 || D > most_devices || K > most_types || NR > most_nr || gt.maxin > 2 || gt.maxout > 2) return false;
    if (kp.space != kSampledStrict && kp.space != kSampledRepair) return false;
    size_t distinct = 0;
    for (int i = 0; i < K; i++) distinct += in[i].size();
    if (distinct != p.dep_src.size() || span_max > 30000) return false;
    if ((int64_t)kp.UB * (std::max(9, gt.retry_tries) + 1) > 65535) return false;
    constexpr int rows = 3, words = 8, mem_at = 16;
    constexpr uint32_t row = kWave * 4, half = row / 2, ts = 128;
    // (the layout below overwrites that of words by type, so nothing is refused from here on)
    static_assert(words * ts + most_types * 16 + 3 * row + (2 * most_devices + most_types * 3 * most_nr + 2 * most_nr) * half + most_types / 4 * row <= 64 * 1024 - row &&
                  words * ts + most_types * 16 + 2 * row + most_devices * rows * row <= 64 * 1024 - row,
                  "tables and the rows of the build and of the sweeps fit");
    uint32_t at = (uint32_t)words * ts;
    gt.sw = at; at += (uint32_t)K * 16;
    gt.ntab = (int)(at / 4);
    at = (at + row - 1) / row * row;
    gt.slot_rows = at; at += row;
    gt.rec = at;
    const uint32_t build_end = at + (uint32_t)(D * rows) * row;
    gt.state = at; at += (uint32_t)kp.nslots * half;
    gt.prev = at; at += (uint32_t)D * half;
    const uint32_t apart = at;
    for (int r = 0; r < kp.ntok; r++) if (kp.ring_kept[r] == kp.ring_base[r]) at += (uint32_t)NR * half;
    gt.apart_rows = (int)((at - apart) / half);
    // (a ring that nobody reads: a type without consumers is N_R micro-batches from its lead on, which is 0 unless it is fixed)
    gt.strash = at; at += (uint32_t)(kp.has_fixed ? 2 * NR : NR) * half;
    at = (at + row - 1) / row * row;
    gt.leads = at; at += (uint32_t)((kp.ntok + 3) / 4) * row;
    gt.lds_bytes = std::max(build_end, at);
    memset(gt.tab, 0, sizeof gt.tab);
    gt.apart = 1;
    for (uint32_t r = 0, row_at = (apart - gt.state) / half; r < (uint32_t)kp.ntok; r++)
        if (kp.ring_kept[r] == kp.ring_base[r]) { gt.ring[r] = (uint32_t)kp.ring_base[r] | row_at << 16; row_at += (uint32_t)NR; }
    gt.codes = 3;
    gt.np = 0;
    std::vector<int> code(K, 0);
    for (int d = 0; d < D; d++)
        for (int y = 0; y < kp.ntd[d]; y++) code[kp.type_of[d] >> (8 * y) & 0xFFu] = 2 * d + y;
    auto dev = [&](int g) -> int { return code[g] >> 1; };
    auto wait_at = [&](int g, int slot) -> int { return 10 * (code[g] & 1) + 5 * slot; };
    auto slot_of = [&](int g, int h) -> int { return (int)(std::find(in[h].begin(), in[h].end(), g) - in[h].begin()); };
    auto word = [&](int w, int c) -> uint32_t & { return gt.tab[((uint32_t)w * ts) / 4 + (uint32_t)c]; };
    auto rec_row = [&](int d, int r) -> uint32_t { return gt.rec + (uint32_t)(d * rows + r) * row; };
    gt.free0 = gt.free1 = 0;
    for (int g = 0; g < K; g++) {
        const int c = code[g];
        for (int s = (int)in[g].size(); s < 2; s++) {
            (s ? gt.free1 : gt.free0) |= 1u << c;
            gt.waits[dev(g)] += (uint32_t)(NR + 1) << wait_at(g, s);                  // (never used up)
        }
        word(0, c) = 0u - (1u << wait_at(g, 0)) - (1u << wait_at(g, 1));
        word(1, c) = (uint32_t)p.m[g] << mem_at;
        for (int k = 0; k < 2; k++) {
            uint32_t to = rec_row(dev(g), 1), inc = 0;
            if (k < (int)outs[g].size()) {
                const int h = outs[g][k], s = slot_of(g, h);
                word(2 + s, c) |= 1u << code[h];
                if (dev(h) == dev(g)) word(0, c) += 1u << wait_at(h, s);
                else { to = rec_row(dev(h), 1); inc = 1u << wait_at(h, s); }
            }
            word(4 + 2 * k, c) = to | (k ? 0u : ((uint32_t)g * 8u + ((uint32_t)(NR - 1) << 9)) << 16);
            word(5 + 2 * k, c) = inc;
        }
        auto ring_address = [&](int i) -> uint32_t { return gt.state + (uint32_t)kp.tokbase[i] * half; };
        const uint32_t to = kp.tokbase[g] != kNoRing ? ring_address(g) : gt.strash;
        uint32_t from[2];
        for (int s = 0; s < 2; s++) from[s] = in[g].empty() ? to : ring_address(in[g][s < (int)in[g].size() ? s : 0]);
        uint32_t *e = &gt.tab[gt.sw / 4 + 4 * g];
        e[0] = (uint32_t)p.t[g];
        e[1] = (gt.state + (uint32_t)dev(g) * half) | to << 16;
        e[2] = from[0] | from[1] << 16;
        uint32_t *l = gt.links[g];
        l[0] = rec_row(dev(g), 1);
        l[1] = (uint32_t)(4 * (c & 1)) | (uint32_t)c << 8;
        l[2] = 0;
        l[3] = (uint32_t)p.m[g] << mem_at;
    }
    gt.nedge = 0;
    for (int b = 0; b < K; b++)
        for (size_t s = 0; s < in[b].size(); s++)
            gt.edge[gt.nedge++] = (uint32_t)in[b][s] | (uint32_t)b << 8 | (uint32_t)wait_at(b, (int)s) << 16 | (uint32_t)s << 24;
    for (int r = 0; r < kp.ntok; r++) {
        const int g = kp.ring_head[r];
        gt.head[r] = rec_row(dev(g), 2) | (uint32_t)(4 * (code[g] & 1)) << 16 | 4u << 24;
    }
    gt.ok = 1;
    return true;
}

// Tables of the graph kernel (GraphTab).  Leaves ok = 0 where the problem is outside what they hold: more than kGraphOut
// consumers or the fields of a type's word producers of one type, a type without any dependency, more than kGraphTp types
// on several devices, memory prefixes beyond 16 bits, an LDS need beyond 64 KB, and where the general kernel is faster.
static void graph_tables(const tessel_problem &p, GraphTab &gt)
{
    memset(&gt, 0, sizeof gt);
    const KParams &kp = p.kp;
    const int D = kp.D, K = kp.K, NR = kp.NR;
    if (!kp.dag) return;
    // Exhaustive spaces on up to 8 devices and 32 types, where most candidates fall to their decode or their first blocks and the
    // graph kernel's tables and the launch over its list are dear.  Against the general kernel (scores of 8 to 500,003 candidates,
    // random graphs, fans, K-shape, diamond; geometric means over ranges of sizes): blocks on several devices 0.98 to 1.35 of its
    // time, windows of one micro-batch 1.04 to 1.14, FACTORIAL 0.83 to 1.09: left to it.  CANONICAL 0.82 to 0.95, though
    // up to 5 us longer where no candidate of a short call gets past its first blocks.  (More devices or types: 0.2 to 0.8 in both, as above
    // 3 us longer at worst.)
    const bool exhaustive = kp.space == kFactorial || kp.space == kCanonical;
    if (exhaustive && D <= kMaxD && K <= kMaxK && (kp.tp || NR == 1 || kp.space == kFactorial)) return;
    int most = 0;
    for (int d = 0; d < D; d++) most = std::max(most, kp.ntd[d]);
    gt.np = most <= 2 ? 1 : most <= 4 ? 2 : 3;
    // distinct dependencies, by consumer and by producer
    std::vector<std::vector<int>> in(K), outs(K);
    for (size_t e = 0; e < p.dep_src.size(); e++) {
        const int a = p.dep_src[e], b = p.dep_dst[e];
        if (std::find(in[b].begin(), in[b].end(), a) == in[b].end()) { in[b].push_back(a); outs[a].push_back(b); }
    }
    for (int i = 0; i < K; i++) {
        if (in[i].empty() && outs[i].empty()) return;
        gt.maxout = std::max(gt.maxout, (int)outs[i].size());
        gt.maxin = std::max(gt.maxin, (int)in[i].size());
    }
    if (gt.maxout > kGraphOut || gt.maxin > kGraphIn) return;
    gt.chain = gt.maxout <= 1 && gt.maxin <= 1;
    // the word of a type: next micro-batch (up to 2 N_R - 1) on top, fields with a guard bit below
    int bits = 1;
    while ((1 << bits) <= 2 * NR - 1) bits++;
    const int f = bits + 1, fields = (32 - bits) / f;
    if (1 + gt.maxin > fields) return;
    gt.mushift = 32 - bits;
    for (int s = 0; s < fields; s++) { gt.add |= ((1u << bits) - 1u) << (f * s); gt.guard |= 1u << (f * s + bits); }
    long span_max = 0;
    for (int d = 0; d < D; d++) {
        long span = 0;
        for (int i = 0; i < K; i++) if (p.mask[i] >> d & 1u) span += std::labs((long)p.m[i]) * (2 * NR - 1);
        span_max = std::max(span_max, span);
    }
    if (span_max > 30000 || (int64_t)kp.UB * 64 >= (int64_t)1 << 31) return;
    // the dependencies for the sampled leads, consumers before producers
    for (int k = 0; k < K; k++) {
        const int i = kp.rtopo[k], from = gt.nlead;
        for (int e = 0; e < kp.ndeps; e++)
            if (kp.dsrc[e] == i)
                gt.lead_edge[gt.nlead++] = (uint32_t)i | (uint32_t)kp.ddst[e] << 8 | (uint32_t)e << 16 | (uint32_t)(kp.dcross[e] != 0) << 24;
        if (gt.nlead > from) { gt.lead_edge[from] |= 1u << 25; gt.lead_edge[gt.nlead - 1] |= 1u << 26; }
    }
    for (int b = 0; b < K; b++)
        for (size_t s = 0; s < in[b].size(); s++)
            gt.edge[gt.nedge++] = (uint32_t)in[b][s] | (uint32_t)b << 8 | (uint32_t)(f * (1 + (int)s)) << 16;
    gt.first_tries = std::min(kGraphTries, kp.dag_tries);
    // (every period seen settled within eight sweeps or never; a wave waits for its slowest lane)
    gt.retry_tries = kp.dag_tries + kp.dag_tries / 2;
    gt.nwords = ((kp.total + 1) / 2 + 3) / 4 * 4;
    gt.meta = 3 + (kp.ntok + 3) / 4;
    for (int d = 0; d < D; d++) gt.busy |= (kp.ntd[d] > 0 ? 1u : 0u) << d;
    for (int r = 0; r < kp.ntok; r++) gt.ring[r] = (uint32_t)kp.ring_base[r] | (uint32_t)kp.ring_kept[r] << 16;
    // LDS: code tables, sweep tables, tables of types on several devices, slot rows, then build and sweep state in one place
    const int cw = 2 + 2 * gt.maxout;                       // words of a code
    const uint32_t row = kWave * 4;
    gt.code_bytes = (uint32_t)cw * 4;
    uint32_t at = ((uint32_t)D << gt.np) * gt.code_bytes;
    const int pairs = gt.chain && !kp.tp ? 0 : (gt.maxin + 1) / 2;
    gt.sw = at; at += (uint32_t)K * 8;
    gt.swp = at; at += (uint32_t)(pairs * K) * 4;
    gt.init = at; at += (uint32_t)K * 4;
    for (int i = 0; i < K; i++) {
        uint32_t w = (uint32_t)NR;
        for (int s = (int)in[i].size(); s < fields - 1; s++) w |= 1u << (f * (1 + s));
        gt.tab[gt.init / 4 + i] = w;
    }
    gt.dev = at; at += (uint32_t)D * 4;
    for (int d = 0; d < D; d++) gt.tab[gt.dev / 4 + d] = (uint32_t)kp.ntd[d];
    std::vector<int> tp_no(K, -1);
    if (kp.tp) {
        for (int i = 0; i < K; i++) if (p.mask[i] & (p.mask[i] - 1)) tp_no[i] = gt.ntp++;
        if (gt.ntp > kGraphTp) return;
        gt.tpm = at; at += kMaxKW * 4;
        gt.tpi = at; at += (kMaxKW + kGraphTp) * 4;
        gt.tps = at; at += (uint32_t)gt.ntp * 32 * 4;
        gt.smask = at; at += 32 * 4;
    }
    gt.ntab = (int)(at / 4);
    at = (at + row - 1) / row * row;
    gt.slot_rows = at; at += row;
    const uint32_t base = at;
    gt.rec = at; at += (uint32_t)D * (gt.np + 2) * row;
    gt.wrow = at; at += (uint32_t)K * row;
    gt.trash = at; at += row;
    const uint32_t build_end = at;
    at = base;
    gt.state = at; at += (uint32_t)kp.nslots * row;
    gt.prev = at; at += (uint32_t)D * row;
    gt.strash = at; at += row;
    gt.leads = at; at += (uint32_t)((kp.ntok + 3) / 4) * row;
    gt.lds_bytes = std::max(build_end, at);
    if (gt.lds_bytes > 64 * 1024 - row) return;             // (16-bit LDS addresses, eight-bit row numbers)
    // (test knob: 1 = a word a type for all problems, 0 = for none, and masks by code for chains alone (the others left to the general kernel))
    const char *words = getenv("TESSEL_GRAPH_WORDS");
    if (!(words && words[0] == '1') && code_tables(p, gt, in, outs, span_max)) return;
    if (!words && graph_code_tables(p, gt, in, outs, span_max)) return;
    if (words && words[0] == '0') return;
    for (int r = 0; r < kp.ntok; r++) gt.head[r] = gt.wrow + (uint32_t)kp.ring_head[r] * row;
    auto type_at = [&](int d, int y) -> int { return (int)((y < 4 ? kp.type_of[d] >> (8 * y) : kp.type_of_hi[d] >> (8 * (y - 4))) & 0xFFu); };
    auto symbol_on = [&](int g, int d) -> int { for (int y = 0; y < kp.ntd[d]; y++) if (type_at(d, y) == g) return y; return 0; };
    auto lowest = [&](int g) -> int { return __builtin_ctz(p.mask[g]); };
    for (int d = 0; d < D; d++)
        for (int y = 0; y < kp.ntd[d]; y++) {
            const int g = type_at(d, y), c = ((d << gt.np) + y) * cw;
            gt.tab[c] = ((uint32_t)p.m[g] << 16) | (((gt.wrow + (uint32_t)g * row) / row) << 8) | (tp_no[g] >= 0 ? 64u : 0u) | (uint32_t)g;
            uint32_t dec = (1u << gt.mushift) - 1u;
            for (size_t s = 0; s < in[g].size(); s++) dec -= 1u << (f * (1 + (int)s));
            gt.tab[c + 1] = dec;
            for (int k = 0; k < gt.maxout; k++) {
                uint32_t c0, c1 = 0;
                if (k < (int)outs[g].size()) {
                    const int h = outs[g][k], dh = lowest(h);
                    const int slot = (int)(std::find(in[h].begin(), in[h].end(), g) - in[h].begin());
                    c0 = (gt.rec + (uint32_t)(dh * (gt.np + 2) + gt.np + 1) * row) << 16 | ((gt.wrow + (uint32_t)h * row) / row) << 8 |
                         (uint32_t)dh << 3 | (uint32_t)symbol_on(h, dh);
                    c1 = 1u << (f * (1 + slot));
                } else
                    c0 = (gt.rec + (uint32_t)(d * (gt.np + 2) + gt.np + 1) * row) << 16 | (gt.trash / row) << 8 | (uint32_t)d << 3;
                gt.tab[c + 2 + 2 * k] = c0;
                gt.tab[c + 3 + 2 * k] = c1;
            }
        }
    // rings: a type of a shared stretch reads and writes the stretch's; a type with no producer reads its own, where its
    // micro-batch has not been written; a type nobody consumes writes nothing (chains: the stretch's ring, read by nobody then)
    std::vector<uint32_t> ring(K, 0);
    auto ring_address = [&](int g) -> uint32_t { return gt.state + (uint32_t)kp.tokbase[g] * row; };
    for (int g = 0; g < K; g++) {
        const bool own = kp.tokbase[g] != kNoRing;
        uint32_t to = own ? ring_address(g) : gt.strash;
        if (gt.chain && !own) to = ring_address(in[g][0]);
        gt.tab[gt.sw / 4 + 2 * g] = (uint32_t)p.t[g] | (own ? 1u << 31 : 0u);
        gt.tab[gt.sw / 4 + 2 * g + 1] = (gt.state + (uint32_t)lowest(g) * row) | to << 16;
        for (int k = 0; k < pairs; k++) {
            auto from = [&](int s) -> uint32_t { return in[g].empty() ? to : ring_address(s < (int)in[g].size() ? in[g][s] : in[g][0]); };
            gt.tab[gt.swp / 4 + k * K + g] = from(2 * k) | from(2 * k + 1) << 16;
        }
    }
    if (kp.tp)
        for (int g = 0; g < K; g++) {
            if (tp_no[g] < 0) {
                gt.tab[gt.smask / 4 + lowest(g)] |= 1u << symbol_on(g, lowest(g));
                continue;
            }
            const uint32_t info = (uint32_t)(6 * tp_no[g]) | (uint32_t)lowest(g) << 8 | (uint32_t)__builtin_popcount(p.mask[g]) << 16;
            gt.tab[gt.tpm / 4 + g] = p.mask[g];
            gt.tab[gt.tpi / 4 + g] = info;
            gt.tab[gt.tpi / 4 + kMaxKW + tp_no[g]] = info;
            for (int d = 0; d < D; d++) if (p.mask[g] >> d & 1u) gt.tab[gt.tps / 4 + tp_no[g] * 32 + d] = (uint32_t)symbol_on(g, d);
        }
    gt.ok = 1;
}

// Sizes of the fast kernel's tables by rank for the CANONICAL space (KParams::ranked), in entries; false where neither is
// made: the kernel then unranks symbol by symbol.
static bool ranked_sizes(tessel_problem &p, size_t &orders, size_t &leadrows)
{
    KParams &kp = p.kp;
    orders = leadrows = 0;
    if (!kp.fast_ok || p.nlead > kRankedLeads) return false;
    size_t by_types[kMaxLT + 1] = {0};
    for (int d = 0; d < kp.D; d++) {
        if (kp.cdev[d] > kRankedOrders) return false;
        by_types[kp.ntd[d]] = kp.cdev[d];
    }
    // (at most 0.9 of the 1 MiB the workspace has for tables)
    for (int n = 0; n <= kMaxLT; n++) { kp.order_at[n] = (uint32_t)orders; orders += by_types[n]; }
    leadrows = p.nlead * kLeadRow;
    return true;
}

// Every order of a device in rank order (lexicographic), and for every lead vector what the build makes of it, written
// where the workspace's copy of them is made up (zeros so far).  Every handle pays for them: 16 us for 2,520 orders of four types
// (std::next_permutation and vectors of their own: 58), 0.1 ms for 3,675 lead vectors of eight types (0.38).
static void fill_ranked(const tessel_problem &p, uint64_t *orders, uint32_t *leadrows)
{
    const KParams &kp = p.kp;
    bool done[kMaxLT + 1] = {false};
    for (int d = 0; d < kp.D; d++) {
        if (done[kp.ntd[d]]) continue;
        done[kp.ntd[d]] = true;
        uint64_t *out = orders + kp.order_at[kp.ntd[d]];
        const int types = kp.ntd[d], len = types * kp.NR;
        int left[kMaxLT];
        for (int y = 0; y < types; y++) left[y] = kp.NR;
        auto extend = [&](auto &self, int pos, uint64_t planes) -> void {
            if (pos == len) { *out++ = planes; return; }
            for (int y = 0; y < types; y++)
                if (left[y] > 0) {
                    left[y]--;
                    self(self, pos + 1, planes | (uint64_t)(y & 1) << pos | (uint64_t)(y >> 1) << (32 + pos));
                    left[y]++;
                }
        };
        extend(extend, 0, 0);
    }
    struct Code { int g, a, word, shift; } code[kMaxK];
    int codes = 0;
    uint32_t absent[4] = {~0u, ~0u, ~0u, ~0u};                       // 15 where there is no type: a chain's first block never waits either
    for (int d = 0; d < kp.D; d++)
        for (int y = 0; y < kp.ntd[d]; y++) {
            const int c = 4 * d + y, g = (int)((kp.type_of[d] >> (8 * y)) & 0xFFu), a = kp.pred[g];
            code[codes++] = Code{g, a, c / 8, 4 * (c % 8)};
            if (a >= 0) absent[c / 8] &= ~(15u << (4 * (c % 8)));
        }
    for (uint64_t v = 0; v < p.nlead; v++) {
        const int8_t *lead = p.leadtab.data() + v * (uint64_t)kp.K;
        uint32_t *row = leadrows + v * kLeadRow;
        for (int w = 0; w < 4; w++) row[4 + w] = absent[w];
        for (int k = 0; k < codes; k++) {
            const Code &c = code[k];
            const uint32_t wait = c.a < 0 ? 15u : (uint32_t)(lead[c.a] - lead[c.g]);
            row[c.word] |= (uint32_t)lead[c.g] << c.shift;
            row[4 + c.word] |= wait << c.shift;
            row[8] |= (wait ? 1u : 0u) << (8 * c.word + c.shift / 4);
        }
    }
}

// The pairs of devices that a dependency joins (KParams::npairs), their tables behind the others in the `room` that is left.
static void list_pairs(tessel_problem &p, size_t room)
{
    KParams &kp = p.kp;
    kp.npairs = 0;
    kp.pair_words = kp.pair_bits = 0;
    bool joined[kMaxD][kMaxD] = {};
    for (int g = 0; g < kp.K; g++)
        if (kp.pred[g] >= 0) {
            const int a = __builtin_ctz(p.mask[kp.pred[g]]), b = __builtin_ctz(p.mask[g]);
            if (a != b) joined[std::min(a, b)][std::max(a, b)] = true;
        }
    uint64_t words = 0, bits = 0;
    for (int d = 0; d < kp.D; d++)
        for (int e = d + 1; e < kp.D; e++) {
            const uint64_t both = kp.cdev[d] * kp.cdev[e];          // (16,384 orders each at most)
            if (!joined[d][e] || both <= 1) continue;
            kp.pair_of[kp.npairs][0] = (uint8_t)d; kp.pair_of[kp.npairs][1] = (uint8_t)e;
            kp.pair_at[kp.npairs++] = (uint32_t)words;
            words += (both + 63) / 64 * 2; bits += both;
            if (words * 4 > room) { kp.npairs = 0; return; }
        }
    kp.pair_words = (uint32_t)words; kp.pair_bits = (uint32_t)bits; kp.pair_room = (uint32_t)(room / 4);
}

extern "C" int tessel_problem_create(const tessel_problem_desc *desc, tessel_problem **out)
{
    if (!desc || !out) return TESSEL_E_INVALID_ARG;
    *out = nullptr;
    const int D = desc->num_devices, K = desc->num_block_types, NR = desc->nr;
    if (D < 1 || K < 1 || NR < 1 || desc->num_deps < 0 || !desc->time || !desc->mem || !desc->dev_mask ||
        (desc->num_deps > 0 && (!desc->dep_src || !desc->dep_dst)) || desc->space < 0 || desc->space > 3 ||
        desc->lead_step_q16 > 65536u)
        return TESSEL_E_INVALID_ARG;
    if (D > kMaxDW) return TESSEL_E_UNSUPPORTED;
    for (int i = 0; i < K; i++)
        if (desc->time[i] < 1 || desc->dev_mask[i] == 0 || (D < 32 && (desc->dev_mask[i] >> D))) return TESSEL_E_INVALID_ARG;
    for (int e = 0; e < desc->num_deps; e++)
        if (desc->dep_src[e] < 0 || desc->dep_src[e] >= K || desc->dep_dst[e] < 0 || desc->dep_dst[e] >= K ||
            desc->dep_src[e] == desc->dep_dst[e])
            return TESSEL_E_INVALID_ARG;
    if (desc->fixed_leads) {
        if (desc->space == TESSEL_SPACE_FACTORIAL) return TESSEL_E_INVALID_ARG;
        for (int i = 0; i < K; i++) if (desc->fixed_leads[i] < 0 || desc->fixed_leads[i] >= NR) return TESSEL_E_INVALID_ARG;
        for (int e = 0; e < desc->num_deps; e++)
            if (desc->fixed_leads[desc->dep_src[e]] < desc->fixed_leads[desc->dep_dst[e]]) return TESSEL_E_INVALID_ARG;
    }
    // acyclic?
    {
        std::vector<int> indeg(K, 0), done(K, 0);
        for (int e = 0; e < desc->num_deps; e++) indeg[desc->dep_dst[e]]++;
        int n = 0;
        for (bool again = true; again;) {
            again = false;
            for (int i = 0; i < K; i++) if (!done[i] && indeg[i] == 0) {
                done[i] = 1; n++; again = true;
                for (int e = 0; e < desc->num_deps; e++) if (desc->dep_src[e] == i) indeg[desc->dep_dst[e]]--;
            }
        }
        if (n != K) return TESSEL_E_BAD_DEP;
    }
    for (int d = 0; d < D; d++) {
        int net = 0;
        for (int i = 0; i < K; i++) if (desc->dev_mask[i] >> d & 1u) net += desc->mem[i];
        if (net != 0) return TESSEL_E_UNBALANCED_MEMORY;
    }
    // limits of the kernels
    if (K > kMaxKW || NR > kMaxNRW) return TESSEL_E_UNSUPPORTED;
    std::vector<int> indeg(K, 0), outdeg(K, 0);
    for (int e = 0; e < desc->num_deps; e++) { outdeg[desc->dep_src[e]]++; indeg[desc->dep_dst[e]]++; }
    // disjoint chains take the fast kernel and the chain path of the general one; any other graph (Sec. III-A allows
    // any acyclic one) the general kernel's path for graphs, which TESSEL_FORCE_DAG=1 also forces on chains (tests)
    bool chains = true;
    for (int i = 0; i < K; i++) if (indeg[i] > 1 || outdeg[i] > 1) chains = false;
    { const char *fd = getenv("TESSEL_FORCE_DAG"); if (fd && fd[0] == '1') chains = false; }
    // more than kMaxD devices or kMaxK block types: the tables by (device, symbol) code of the chain path and of the fast
    // kernel have no room for them; such a problem is scored as a graph, chains or not
    // ... and so is one with more than kMaxLT block types on a device (3-bit symbols; sampled spaces only, at most 32
    // blocks per device and window)
    bool many = false;
    for (int d = 0; d < D; d++) {
        int n = 0;
        for (int i = 0; i < K; i++) n += desc->dev_mask[i] >> d & 1u;
        if (n > kMaxLTW || n * NR > kMaxPos) return TESSEL_E_UNSUPPORTED;
        if (n > kMaxLT) many = true;
    }
    // ... and one with a window of more than kMaxNR micro-batches (8-bit instead of 4-bit counters; sampled spaces only)
    const bool longwin = NR > kMaxNR;
    if ((many || longwin) && desc->space != TESSEL_SPACE_SAMPLED_STRICT && desc->space != TESSEL_SPACE_SAMPLED_REPAIR) return TESSEL_E_UNSUPPORTED;
    const bool wide = D > kMaxD || K > kMaxK || many || longwin;
    if (wide) chains = false;
    if (!chains && desc->num_deps > kMaxDeps) return TESSEL_E_UNSUPPORTED;

    tessel_problem *p = new (std::nothrow) tessel_problem();
    if (!p) return TESSEL_E_INVALID_ARG;
    p->id = g_next_id.fetch_add(1);
    p->t.assign(desc->time, desc->time + K);
    p->m.assign(desc->mem, desc->mem + K);
    p->mask.assign(desc->dev_mask, desc->dev_mask + K);
    p->dep_src.assign(desc->dep_src, desc->dep_src + desc->num_deps);
    p->dep_dst.assign(desc->dep_dst, desc->dep_dst + desc->num_deps);
    KParams &kp = p->kp;
    memset(&kp, 0, sizeof kp);
    kp.D = D; kp.K = K; kp.NR = NR; kp.M = desc->mem_cap; kp.total = K * NR; kp.space = desc->space;
    kp.seed = desc->seed; kp.step_q16 = desc->lead_step_q16;
    kp.has_fixed = desc->fixed_leads != nullptr;
    for (int i = 0; i < K; i++) kp.fixed[i] = desc->fixed_leads ? (uint8_t)desc->fixed_leads[i] : 0;
    for (int i = 0; i < K && i < kMaxK; i++) { kp.pred[i] = -1; kp.succ[i] = -1; }
    for (int e = 0; e < desc->num_deps && chains; e++) {
        int a = desc->dep_src[e], b = desc->dep_dst[e];
        kp.succ[a] = (int8_t)b; kp.pred[b] = (int8_t)a;
        kp.edge_out[a] = (uint8_t)e;
        kp.cross_out[a] = desc->dev_mask[a] != desc->dev_mask[b];
    }
    if (!chains) {
        kp.dag = 1; kp.ndeps = desc->num_deps;
        kp.dag_tries = 8;
        if (const char *env = getenv("TESSEL_DAG_TRIES")) {        // test knob: 0 leaves every period to the bisection
            int v = atoi(env);
            if (v >= 0 && v <= 64) kp.dag_tries = v;
        }
        for (int i = 0; i < K; i++) { kp.t_type[i] = desc->time[i]; kp.mask_type[i] = desc->dev_mask[i]; kp.tokbase[i] = (uint16_t)kNoRing; }
        for (int e = 0; e < desc->num_deps; e++) {
            const int a = desc->dep_src[e], b = desc->dep_dst[e];
            kp.dsrc[e] = (uint8_t)a; kp.ddst[e] = (uint8_t)b; kp.dcross[e] = desc->dev_mask[a] != desc->dev_mask[b];
            kp.predmask[b] |= 1ull << a;
        }
        // End times by micro-batch, 2 N_R slots per ring behind the devices (and for a shared ring N_R more: what the last
        // window boundary left in the ring's lower half, for the comparison at the next one).  A stretch of the graph without branches
        // (a -> b with a's only consumer b and b's only producer a) shares one ring: b reads a's end time of a
        // micro-batch and puts its own in its place, which only b's consumers read.  A chain is one ring.
        {
            std::vector<int> head(K), next_in(K, -1);
            for (int i = 0; i < K; i++) head[i] = i;
            for (int e = 0; e < desc->num_deps; e++) {
                const int a = desc->dep_src[e], b = desc->dep_dst[e];
                bool twice = false;                          // (a dependency listed twice counts once)
                for (int f = 0; f < e; f++) if (desc->dep_src[f] == a && desc->dep_dst[f] == b) twice = true;
                int outs = 0, ins = 0;
                for (int f = 0; f < desc->num_deps; f++) {
                    bool seen = false;
                    for (int h = 0; h < f; h++) if (desc->dep_src[h] == desc->dep_src[f] && desc->dep_dst[h] == desc->dep_dst[f]) seen = true;
                    if (seen) continue;
                    outs += desc->dep_src[f] == a; ins += desc->dep_dst[f] == b;
                }
                if (!twice && outs == 1 && ins == 1) next_in[a] = b;
            }
            std::vector<char> inner(K, 0);
            int slots = 0;
            for (int i = 0; i < K; i++) if (next_in[i] >= 0) inner[next_in[i]] = 1;
            for (int i = 0; i < K; i++) {
                if (inner[i]) continue;                       // i starts a stretch
                bool consumed = false;
                for (int g = i; g >= 0; g = next_in[g]) consumed = consumed || outdeg[g] > 0;
                if (!consumed) continue;
                const int base = D + slots;
                const bool shared = next_in[i] >= 0;
                kp.ring_head[kp.ntok] = (uint8_t)i;
                kp.ring_base[kp.ntok] = (uint16_t)base;
                kp.ring_kept[kp.ntok] = (uint16_t)(shared ? base + 2 * NR : base);
                for (int g = i; g >= 0; g = next_in[g]) if (outdeg[g] > 0) kp.tokbase[g] = (uint16_t)base;
                kp.ntok++;
                slots += (shared ? 3 : 2) * NR;
            }
            kp.nslots = D + slots;
        }
        // consumers before producers
        std::vector<int> left(outdeg), done(K, 0);
        int n = 0;
        for (bool again = true; again;) {
            again = false;
            for (int i = 0; i < K; i++) if (!done[i] && left[i] == 0) {
                done[i] = 1; kp.rtopo[n++] = (uint8_t)i; again = true;
                for (int e = 0; e < desc->num_deps; e++) if (desc->dep_dst[e] == i) left[desc->dep_src[e]]--;
            }
        }
    }
    // chains and their token slots; reverse topological order = walk every chain from its end
    std::vector<int> path_of(K, 0);
    int npaths = 0, nrt = 0;
    if (chains) {
        for (int i = 0; i < K; i++) if (kp.pred[i] < 0) {
            for (int g = i; g >= 0; g = kp.succ[g]) path_of[g] = npaths;
            npaths++;
        }
        for (int i = 0; i < K; i++) if (kp.succ[i] < 0)
            for (int g = i; g >= 0; g = kp.pred[g]) kp.rtopo[nrt++] = (uint8_t)g;
        kp.npaths = npaths;
        kp.nslots = D + npaths * 2 * NR;
        kp.nsweeps = D + npaths * NR + 1;
        if (kp.nslots > 63 || kp.nsweeps - 1 > 24) { delete p; return TESSEL_E_UNSUPPORTED; }
    } else {
        kp.npaths = 0;
        kp.nsweeps = D + 1;                       // (only sizes the register arrays of the chain path, unused here)
        // state and program of a workgroup must fit the LDS a kernel may ask for
        // (problems too wide for the other paths keep both in global memory when they have to)
        if (!wide && (size_t)4 * kMaxK * 4 + (size_t)kp.nslots * kWave * 4 + (size_t)K * NR * kWave * 2 > 64 * 1024) { delete p; return TESSEL_E_UNSUPPORTED; }
    }
    int sumt = 0;
    for (int i = 0; i < K; i++) {
        if (desc->time[i] > (1 << 20)) { delete p; return TESSEL_E_TOOBIG; }
        sumt += desc->time[i];
    }
    kp.UB = NR * sumt;
    // the period kernel multiplies (sweeps * UB) by a sweep count
    if ((int64_t)kp.UB * kp.nsweeps * kp.nsweeps >= (int64_t)1 << 31) { delete p; return TESSEL_E_TOOBIG; }
    kp.LB = 0;
    for (int d = 0; d < kMaxDW; d++) kp.type_of[d] = kp.type_of_hi[d] = 0xFFFFFFFFu;
    kp.many = many;
    for (int d = 0; d < kMaxD; d++) { kp.pred_of[d] = 0xFFFFFFFFu; kp.mask_of[d] = kp.tok_of[d] = kp.home_of[d] = 0; }
    std::vector<int> home(K, -1);
    for (int d = 0; d < D; d++) {
        int n = 0, busy = 0;
        for (int i = 0; i < K; i++) if (desc->dev_mask[i] >> d & 1u) {
            if (n >= kMaxLTW) { delete p; return TESSEL_E_UNSUPPORTED; }
            if (home[i] < 0) home[i] = d * 4 + n;
            if (n < 4) kp.type_of[d] = (kp.type_of[d] & ~(0xFFu << (8 * n))) | ((uint32_t)i << (8 * n));
            else kp.type_of_hi[d] = (kp.type_of_hi[d] & ~(0xFFu << (8 * (n - 4)))) | ((uint32_t)i << (8 * (n - 4)));
            if (!wide) {
                uint32_t pr = kp.pred[i] < 0 ? 0xFFu : (uint32_t)kp.pred[i];
                kp.pred_of[d] = (kp.pred_of[d] & ~(0xFFu << (8 * n))) | (pr << (8 * n));
                kp.mask_of[d] |= (desc->dev_mask[i] & 0xFFu) << (8 * n);
                kp.tok_of[d] |= (uint32_t)(D + path_of[i] * 2 * NR) << (8 * n);
                kp.home_of[d] |= (uint32_t)home[i] << (8 * n);
            }
            kp.predmask_of[d][n] = kp.predmask[i];
            kp.m_of[d][n] = desc->mem[i];
            busy += desc->time[i];
            n++;
        }
        kp.ntd[d] = n;
        kp.LB = std::max(kp.LB, NR * busy);
    }
    for (int i = 0; i < K; i++) {
        if (!wide) { kp.t_loc[home[i]] = desc->time[i]; kp.mask_loc[home[i]] = desc->dev_mask[i]; }
        if (desc->dev_mask[i] & (desc->dev_mask[i] - 1)) kp.tp = 1;
    }
    // tables of the fast kernel: single-device blocks, small memory deltas, few slots
    if (!wide) {
        bool ok = chains && kp.nslots <= 32 && kp.nsweeps - 1 <= 24;
        // every (device, local symbol) is a code; a type on several devices has one code per device
        std::vector<std::vector<int>> code_on(K, std::vector<int>(D, -1));
        for (int d = 0; d < D; d++)
            for (int y = 0; y < kp.ntd[d]; y++) code_on[(kp.type_of[d] >> (8 * y)) & 0xFFu][d] = d * 4 + y;
        for (int c = 0; c < kMaxK; c++) kp.home_code[c] = 63;
        for (int i = 0; i < K; i++) {
            uint32_t grp = 0;
            for (int d = 0; d < D; d++) if (code_on[i][d] >= 0) grp |= 1u << code_on[i][d];
            for (int d = 0; d < D; d++) if (code_on[i][d] >= 0) { kp.grp_code[code_on[i][d]] = grp; kp.home_code[code_on[i][d]] = (uint8_t)home[i]; }
            const bool multi = (desc->dev_mask[i] & (desc->dev_mask[i] - 1)) != 0;
            if (multi) { if (kp.ntp < kMaxD) kp.tp_group[kp.ntp++] = grp; else ok = false; }
            if (multi) kp.several |= grp;
        }
        kp.fast_tp = kp.tp;
        kp.tp_all = kp.tp;
        for (int i = 0; i < K; i++)
            if ((desc->dev_mask[i] & (desc->dev_mask[i] - 1)) && desc->dev_mask[i] != (D < 32 ? (1u << D) - 1u : ~0u)) kp.tp_all = 0;
        // the memory prefix of a device is kept in 8 bits: entry (lead <= N_R-1 each) plus N_R occurrences
        for (int d = 0; d < D; d++) {
            long span = 0;
            for (int i = 0; i < K; i++) if (desc->dev_mask[i] >> d & 1u) span += (long)std::abs(desc->mem[i]) * (2 * NR - 1);
            if (span > 120) ok = false;
        }
        for (int i = 0; i < K; i++) if (desc->mem[i] < -127 || desc->mem[i] > 127) ok = false;
        for (int i = 0; i < K; i++) if (desc->time[i] > 65535) ok = false;      // the sweep table keeps t in 16 bits
        for (int i = 0; i < kMaxK; i++) kp.info_loc[i] = 63u | (63u << 6);
        for (int i = 0; i < K && ok; i++) {
            uint32_t su = kp.succ[i] < 0 ? 63u : (uint32_t)home[kp.succ[i]];
            uint32_t pr = kp.pred[i] < 0 ? 63u : (uint32_t)home[kp.pred[i]];
            uint32_t tokbase = (uint32_t)(D + path_of[i] * 2 * NR);
            for (int d = 0; d < D; d++) if (code_on[i][d] >= 0)
                kp.info_loc[code_on[i][d]] = su | (pr << 6) | (tokbase << 12) | (((uint32_t)desc->mem[i] & 0xFFu) << 18);
        }
        for (int k = 0; k < K && ok; k++) {
            int i = kp.rtopo[k];
            uint32_t su = kp.succ[i] < 0 ? 63u : (uint32_t)home[kp.succ[i]];
            kp.chain_tab[k] = (uint32_t)home[i] | (su << 6) | ((uint32_t)(kp.succ[i] < 0 ? 0 : kp.edge_out[i]) << 12) |
                              ((uint32_t)(kp.succ[i] >= 0 && kp.cross_out[i]) << 19) | ((uint32_t)(kp.pred[i] < 0) << 20) |
                              ((uint32_t)i << 21);
        }
        {
            // chain_tab lists every chain from its last block to its first, one chain after the other
            std::vector<int> pos(K, 0);
            for (int d = 0; d < kMaxD; d++) kp.no_pred[d] = 0xFFFFu;
            for (int k = 0; k < K; k++) pos[kp.rtopo[k]] = k;
            for (int i = 0; i < K && ok; i++) {
                uint32_t cum = 0;
                for (int g = i; kp.succ[g] >= 0; g = kp.succ[g]) cum |= 1u << pos[g];
                for (int d = 0; d < D; d++) if (code_on[i][d] >= 0) {
                    kp.cum_code[code_on[i][d]] = cum;
                    if (kp.pred[i] < 0) { kp.first_codes |= 1u << code_on[i][d]; continue; }
                    kp.pred_pos[d] |= (uint32_t)pos[kp.pred[i]] << (8 * (code_on[i][d] & 3));
                    kp.no_pred[d] &= ~(15u << (4 * (code_on[i][d] & 3)));
                }
                if (kp.succ[i] >= 0 && kp.edge_out[i] < kMaxK) kp.dep_bit[kp.edge_out[i]] = kp.cross_out[i] ? 1u << pos[i] : 0u;
            }
            if (desc->num_deps > kMaxK) ok = false;
        }
        for (int d = 0; d < D; d++) {
            kp.vtab[d] = (uint32_t)d | (1u << 6) | ((uint32_t)(kp.ntd[d] > 0) << 17);
            for (int y = 0; y < kp.ntd[d]; y++) kp.mpack[d] |= ((uint32_t)kp.m_of[d][y] & 0xFFu) << (8 * y);
        }
        int v = D, path = 0;
        for (int i = 0; i < K && ok; i++) if (kp.pred[i] < 0) {
            for (int j = 0; j < NR; j++, v++)
                if (v < 24) kp.vtab[v] = (uint32_t)(D + path * 2 * NR + j) | ((uint32_t)home[i] << 7) | ((uint32_t)j << 13);
            path++;
        }
        kp.fast_ok = ok;
        kp.eigen_tries = kFirstPassTries;
        kp.retry_tries = kRetryTries;
        if (const char *env = getenv("TESSEL_EIGEN_TRIES")) {      // test knobs: force candidates onto the longer search
            int v = atoi(env);
            if (v >= 0 && v <= kMostTries) kp.eigen_tries = v;
        }
        if (const char *env = getenv("TESSEL_RETRY_TRIES")) {      // ... and from there to the general kernel
            int v = atoi(env);
            if (v >= 0 && v <= kMostTries) kp.retry_tries = v;
        }
    }
    // candidate count and the tables of the exhaustive spaces
    if (desc->space == TESSEL_SPACE_FACTORIAL) {
        kp.fact[0] = 1;
        for (int n = 1; n <= 12; n++) kp.fact[n] = kp.fact[n - 1] * (uint32_t)n;
        unsigned __int128 c = 1;
        for (int d = 0; d < D; d++) {
            int n = kp.ntd[d] * NR;
            if (n > 12) { delete p; return n > 20 ? TESSEL_E_TOOBIG : TESSEL_E_UNSUPPORTED; }
            kp.cdev[d] = kp.fact[n];
            uint64_t list = 0;
            int k = 0;
            for (int y = 0; y < kp.ntd[d]; y++)
                for (int l = 0; l < NR; l++, k++) list |= (uint64_t)((y << 3) | l) << (5 * k);
            kp.init_list[d] = list;
            c *= kp.cdev[d];
            if (c >> 64) { delete p; return TESSEL_E_TOOBIG; }
        }
        p->count = (uint64_t)c;
    } else if (desc->space == TESSEL_SPACE_CANONICAL) {
        if (kp.has_fixed) {
            for (int i = 0; i < K; i++) p->leadtab.push_back((int8_t)desc->fixed_leads[i]);
        } else if (!gen_leads(*p, K, NR, p->leadtab, (kWsTablesMax / 2) / K)) {
            delete p; return TESSEL_E_TOOBIG;
        }
        p->nlead = p->leadtab.size() / K;
        unsigned __int128 c = p->nlead;
        for (int d = 0; d < D; d++) {
            int cnt[kMaxLT];
            for (int y = 0; y < kMaxLT; y++) cnt[y] = y < kp.ntd[d] ? NR : 0;
            kp.cdev[d] = multiset_sequences(cnt, kMaxLT);
            if (!kp.cdev[d]) { delete p; return TESSEL_E_TOOBIG; }
            c *= kp.cdev[d];
            if (c >> 64) { delete p; return TESSEL_E_TOOBIG; }
        }
        p->count = (uint64_t)c;
        const int B = NR + 1;
        p->wtab.resize((size_t)B * B * B * B);
        for (int c0 = 0; c0 < B; c0++) for (int c1 = 0; c1 < B; c1++) for (int c2 = 0; c2 < B; c2++) for (int c3 = 0; c3 < B; c3++) {
            int cnt[4] = {c0, c1, c2, c3};
            p->wtab[(((size_t)c0 * B + c1) * B + c2) * B + c3] = multiset_sequences(cnt, 4);   // 0 only where never needed
        }
    } else {
        if (desc->num_deps > 128) { delete p; return TESSEL_E_UNSUPPORTED; }
        p->count = UINT64_MAX;
    }
    p->result.period = INT_MAX;
    { const char *fg = getenv("TESSEL_FORCE_GENERAL"); p->force_general = fg && fg[0] == '1'; }
    { const char *ml = getenv("TESSEL_MAIL"); p->mail = !(ml && ml[0] == '0'); }
    if (p->force_general) kp.fast_ok = 0;
    // (TESSEL_FAR_MODE chooses between placements of the general kernel's state: it takes the problem then)
    p->graph.ok = 0;
    if (!p->force_general && !getenv("TESSEL_FAR_MODE")) graph_tables(*p, p->graph);
    kp.graph_ok = p->graph.ok; kp.graph_np = p->graph.np; kp.graph_codes = p->graph.codes; kp.graph_chain = p->graph.chain; kp.graph_lds = p->graph.lds_bytes;
    kp.graph_slot_words = (uint32_t)(p->graph.meta + p->graph.nwords);
    if (desc->space == TESSEL_SPACE_CANONICAL) {
        size_t orders, leadrows;
        kp.ranked = ranked_sizes(*p, orders, leadrows);
        const size_t bytes[4] = {p->leadtab.size(), p->wtab.size() * 8, orders * 8, leadrows * 4};
        size_t total = 0;
        for (int k = 0; k < 4; k++) { p->table_at[k] = total; total = (total + bytes[k] + 255) & ~(size_t)255; }
        p->image.resize(kWsTablesOff + total);
        char *tables = p->image.data() + kWsTablesOff;
        memcpy(tables, p->leadtab.data(), bytes[0]);
        memcpy(tables + p->table_at[1], p->wtab.data(), bytes[1]);
        if (kp.ranked) {
            fill_ranked(*p, (uint64_t *)(tables + p->table_at[2]), (uint32_t *)(tables + p->table_at[3]));
            for (int d = 0; d < kp.D; d++) kp.recip[d] = kp.cdev[d] > 1 ? (uint32_t)(((uint64_t)1 << 32) / kp.cdev[d]) : 0u;
            if (!kp.fast_tp) list_pairs(*p, kWsTablesMax - total);
        }
    }
    if (p->image.empty()) p->image.resize(kWsTablesOff);
    kp.graph_at = (uint32_t)kWsGraphOff;                             // (where the tables leave it no room: a copy of its own)
    if (kp.graph_ok) {
        const size_t at = (p->image.size() + 255) & ~(size_t)255, bytes = offsetof(GraphTab, tab) + (size_t)p->graph.ntab * 4;
        if (at + bytes <= kWsTablesOff + kWsTablesMax) {
            p->image.resize(at + bytes);
            memcpy(p->image.data() + at, &p->graph, bytes);
            kp.graph_at = (uint32_t)at;
        }
    }
    *out = p;
    return TESSEL_OK;
}

extern "C" void tessel_problem_destroy(tessel_problem *p)
{
    if (!p) return;
    release_workspaces(p);
    delete p;
}

extern "C" int tessel_candidate_count(const tessel_problem *p, uint64_t *count)
{
    if (!p || !count) return TESSEL_E_INVALID_ARG;
    *count = p->count;
    return TESSEL_OK;
}

static int ensure_device(tessel_problem *p)
{
    if (p->num_cus) return TESSEL_OK;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(p, (int)e);
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return hip_fail(p, (int)e);
    p->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    return TESSEL_OK;
}

static size_t workspace_need(const tessel_problem *p, int num_cus)
{
    return eval_workspace_bytes(p->kp, num_cus, 0);
}

extern "C" int tessel_workspace_bytes(const tessel_problem *p, size_t *bytes)
{
    if (!p || !bytes) return TESSEL_E_INVALID_ARG;
    // sized for the grid the launcher uses on the current device (16 workgroups per compute unit at most); for 512
    // compute units where no device can be asked
    int cus = p->num_cus;
    if (!cus) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
            cus = prop.multiProcessorCount;
        else
            (void)hipGetLastError();
    }
    *bytes = workspace_need(p, cus ? cus : 512);
    return TESSEL_OK;
}

static int range_ok(const tessel_problem *p, uint64_t first, uint64_t count)
{
    if (p->count == UINT64_MAX) return first + count >= first ? TESSEL_OK : TESSEL_E_RANGE;
    if (first > p->count || count > p->count - first) return TESSEL_E_RANGE;
    return TESSEL_OK;
}

// Binds the workspace: parameters, tables and the running best `start` (null: none yet) in one copy.  (Two or three copies and a kernel
// for the record took 15 to 25 us more, most of the way to a new handle's first answer in small spaces.)
static int bind_workspace(tessel_problem *p, void *ws, size_t bytes, hipStream_t st, int max_blocks = 0, const DevResult *start = nullptr)
{
    if (!ws || ((uintptr_t)ws & 255u)) return TESSEL_E_WORKSPACE;
    int rc = ensure_device(p);
    if (rc) return rc;
    if (bytes < eval_workspace_bytes(p->kp, p->num_cus, max_blocks)) return TESSEL_E_WORKSPACE;
    if (p->ws == ws && owns_workspace(p)) return TESSEL_OK;
    char *base = (char *)ws + kWsTablesOff;
    if (p->image.size() > kWsTablesOff + kWsTablesMax) return TESSEL_E_TOOBIG;
    if (p->kp.space == kCanonical) {
        p->kp.leadtab = (const int8_t *)(base + p->table_at[0]);
        p->kp.wtab = (const uint64_t *)(base + p->table_at[1]);
        p->kp.orders = (const uint64_t *)(base + p->table_at[2]);
        p->kp.leadrows = (const uint32_t *)(base + p->table_at[3]);
        p->kp.pair_tab = (uint32_t *)((char *)ws + ((p->image.size() + 255) & ~(size_t)255));
    }
    DevResult none;
    memset(&none, 0, sizeof none);
    none.period = INT_MAX; none.index = ~0ull;
    memcpy(p->image.data() + kWsResultOff, start ? start : &none, sizeof none);
    memcpy(p->image.data() + kWsParamsOff, &p->kp, sizeof(KParams));
    // (without tables up to the end of the parameters)
    const size_t upto = p->image.size() > kWsTablesOff ? p->image.size() : kWsParamsOff + sizeof(KParams);
    hipError_t pe = hipMemcpyAsync(ws, p->image.data(), upto, hipMemcpyHostToDevice, st);
    if (pe != hipSuccess) return hip_fail(p, (int)pe);
    if (p->kp.graph_ok && p->kp.graph_at == kWsGraphOff) {
        pe = hipMemcpyAsync((char *)ws + kWsGraphOff, &p->graph, sizeof(GraphTab), hipMemcpyHostToDevice, st);
        if (pe != hipSuccess) return hip_fail(p, (int)pe);
    }
    p->ws = ws; p->ws_ready = true; p->max_blocks = max_blocks;
    p->comp_ready = false;              // the completion parameters lived in the workspace bound before
    p->ranges.clear();
    p->best_dirty = true;
    p->result.period = INT_MAX;
    take_workspace(p, ws);
    return TESSEL_OK;
}

extern "C" int tessel_eval_candidates(tessel_problem *p, uint64_t first, uint64_t count, void *workspace_dev,
                                      size_t workspace_bytes, void *hip_stream)
{
    if (!p) return TESSEL_E_INVALID_ARG;
    int rc = range_ok(p, first, count);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)hip_stream;
    rc = bind_workspace(p, workspace_dev, workspace_bytes, st);
    if (rc) return rc;
    p->stream = st;
    if (count == 0) return TESSEL_OK;
    p->best_dirty = true;
    if (!p->ranges.empty() && p->ranges.back().first + p->ranges.back().second == first) p->ranges.back().second += count;
    else p->ranges.push_back({first, count});
    int e = launch_eval(p->kp, first, count, workspace_dev, p->num_cus, p->max_blocks, st, p->safe_pieces ? kSafePerLaunch : kMaxPerLaunch);
    return e ? hip_fail(p, e) : TESSEL_OK;
}

// tessel_eval_candidates in the library's own device buffer: no allocation anywhere on the way
extern "C" int tessel_eval_candidates_noalloc(tessel_problem *p, uint64_t first, uint64_t count, void *hip_stream)
{
    if (!p) return TESSEL_E_INVALID_ARG;
    int rc = range_ok(p, first, count);
    if (rc) return rc;
    if (count > TESSEL_NOALLOC_MAX_CANDIDATES) return TESSEL_E_TOOBIG;
    rc = ensure_device(p);
    if (rc) return rc;
    void *ws = nullptr;
    size_t bytes = 0;
    int e = scratch_workspace(&ws, &bytes);
    if (e) return hip_fail(p, e);
    const int blocks = eval_blocks_that_fit(p->kp, p->num_cus, bytes);
    if (blocks < 1) return TESSEL_E_WORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    // (a buffer bound with another grid limit, i.e. by the other entry point, cannot be this one: no rebinding check needed)
    rc = bind_workspace(p, ws, bytes, st, blocks);
    if (rc) return rc;
    p->stream = st;
    if (count == 0) return TESSEL_OK;
    p->best_dirty = true;
    if (!p->ranges.empty() && p->ranges.back().first + p->ranges.back().second == first) p->ranges.back().second += count;
    else p->ranges.push_back({first, count});
    e = launch_eval(p->kp, first, count, ws, p->num_cus, p->max_blocks, st, p->safe_pieces ? kSafePerLaunch : kMaxPerLaunch);
    return e ? hip_fail(p, e) : TESSEL_OK;
}

extern "C" int tessel_score_candidates(tessel_problem *p, uint64_t first, uint64_t count, int32_t *code_dev,
                                       int32_t *peak_dev, void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    if (!p || !code_dev) return TESSEL_E_INVALID_ARG;
    int rc = range_ok(p, first, count);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)hip_stream;
    // the workspace carries the tables of the exhaustive spaces; binding a new one clears the running best
    rc = bind_workspace(p, workspace_dev, workspace_bytes, st);
    if (rc) return rc;
    p->stream = st;
    if (count == 0) return TESSEL_OK;
    int e = launch_score(p->kp, first, count, code_dev, peak_dev, workspace_dev, p->num_cus, p->max_blocks, p->force_general, st);
    return e ? hip_fail(p, e) : TESSEL_OK;
}

extern "C" int tessel_alu_probe(int blocks, int rounds, uint32_t *out_dev, size_t out_bytes, void *hip_stream,
                                uint64_t *lane_ops)
{
    if (blocks < 1 || blocks > (1 << 20) || rounds < 1 || rounds > (1 << 24) || !out_dev) return TESSEL_E_INVALID_ARG;
    if (out_bytes < (size_t)blocks * kProbeThreads * sizeof(uint32_t)) return TESSEL_E_WORKSPACE;
    if (lane_ops) *lane_ops = (uint64_t)blocks * kProbeThreads * (uint64_t)rounds * kProbeLaneOpsPerRound;
    return launch_alu_probe(out_dev, blocks, rounds, hip_stream) ? TESSEL_E_HIP : TESSEL_OK;
}

extern "C" int tessel_reset(tessel_problem *p)
{
    if (!p) return TESSEL_E_INVALID_ARG;
    p->result.period = INT_MAX;
    p->ranges.clear();
    p->best_dirty = true;
    if (!owns_workspace(p)) { p->ws_ready = false; return TESSEL_OK; }     // (another handle's by now: nothing of ours is left in it)
    int e = launch_reset(p->ws, p->stream);
    return e ? hip_fail(p, e) : TESSEL_OK;
}

// ---- host post-processing of the single best candidate ---------------------------------
namespace {

// Difference constraints of the repeated window for the decoded candidate (Eq. 1 [1] and [3] with the window-to-window
// lags): block v starts at least w after block u, of the window `lag` before.  By u, the blocks in an executable
// sequence of one window, so that one pass over `edges` carries a start time through all of it.
struct Edge { int u, v, w, lag; };
struct Window {
    int blocks = 0, most = 0;           // most: no least start time is later (every path visits a block at most once)
    std::vector<Edge> edges;
    std::vector<int> from;              // edges of block u: from[u] .. from[u + 1] - 1
};

// sorts the blocks so that every edge `along` selects goes forward; false: these edges have a cycle
template <class Along>
bool in_sequence(const Window &w, Along along, std::vector<int> &sequence)
{
    std::vector<int> waits(w.blocks, 0);
    for (const Edge &e : w.edges) if (along(e)) waits[e.v]++;
    sequence.clear();
    for (int u = 0; u < w.blocks; u++) if (waits[u] == 0) sequence.push_back(u);
    for (size_t k = 0; k < sequence.size(); k++)
        for (int e = w.from[sequence[k]]; e < w.from[sequence[k] + 1]; e++)
            if (along(w.edges[e]) && --waits[w.edges[e].v] == 0) sequence.push_back(w.edges[e].v);
    return (int)sequence.size() == w.blocks;
}

void sort_edges(Window &w, const std::vector<int> &rank)
{
    std::vector<Edge> by(w.edges.size());
    w.from.assign(w.blocks + 1, 0);
    for (const Edge &e : w.edges) w.from[rank[e.u] + 1]++;
    for (int u = 0; u < w.blocks; u++) w.from[u + 1] += w.from[u];
    std::vector<int> next(w.from.begin(), w.from.end() - 1);
    for (const Edge &e : w.edges) by[next[rank[e.u]]++] = Edge{rank[e.u], rank[e.v], e.w, e.lag};
    w.edges.swap(by);
}

// `rank`: number of block type * N_R + occurrence in the window; false: the device orders cannot be executed
bool make_window(const tessel_problem *p, const Detail &c, Window &w, std::vector<int> &rank)
{
    const int NR = p->kp.NR, K = p->kp.K, D = p->kp.D;
    w.blocks = K * NR; w.most = p->kp.UB;
    for (size_t e = 0; e < p->dep_src.size(); e++) {
        int i = p->dep_src[e], j = p->dep_dst[e], delta = c.leads[i] - c.leads[j];
        for (int q = 0; q < NR; q++) {
            int qp = q - delta;
            w.edges.push_back(qp >= 0 ? Edge{i * NR + qp, j * NR + q, p->t[i], 0} : Edge{i * NR + qp + NR, j * NR + q, p->t[i], 1});
        }
    }
    for (int d = 0; d < D; d++) {
        std::vector<int> occ(K, 0), nodes;
        for (int k = 0; k < c.order_len[d]; k++) { int g = c.orders[d][k]; nodes.push_back(g * NR + occ[g]++); }
        for (size_t k = 0; k + 1 < nodes.size(); k++) w.edges.push_back(Edge{nodes[k], nodes[k + 1], p->t[nodes[k] / NR], 0});
        if (!nodes.empty()) w.edges.push_back(Edge{nodes.back(), nodes.front(), p->t[nodes.back() / NR], 1});
    }
    rank.resize(w.blocks);
    std::vector<int> sequence;
    for (int u = 0; u < w.blocks; u++) rank[u] = u;
    sort_edges(w, rank);
    if (!in_sequence(w, [](const Edge &e) { return e.lag == 0; }, sequence)) return false;
    for (int k = 0; k < w.blocks; k++) rank[sequence[k]] = k;
    sort_edges(w, rank);
    return true;
}

// the least non-negative start times at period T; false: there are none, some cycle takes longer than T per window
bool least_starts(const Window &w, int T, std::vector<int> &s)
{
    std::vector<int> by(w.blocks, -1), mark(w.blocks);
    s.assign(w.blocks, 0);
    for (int pass = 0; pass <= w.blocks; pass++) {
        bool changed = false;
        for (const Edge &e : w.edges) {
            const int v = s[e.u] + e.w - e.lag * T;
            if (v <= s[e.v]) continue;
            if (v > w.most) return false;
            s[e.v] = v; by[e.v] = e.u; changed = true;
        }
        if (!changed) return true;
        // a block that owes its start time to itself: that cycle goes on for ever
        std::fill(mark.begin(), mark.end(), -1);
        for (int u = 0; u < w.blocks; u++) {
            int v = u;
            while (v >= 0 && mark[v] < 0) { mark[v] = u; v = by[v]; }
            if (v >= 0 && mark[v] == u) return false;
        }
    }
    return false;
}

// Whether T is the least period, worked out without the kernels' sweeps: there are start times at T, and either some cycle of
// constraints is tight under them, so that it takes T per window exactly (times are positive: such a cycle
// crosses a window boundary), or there are no start times at T - 1 (a ratio that is no whole number, rounded up).
bool is_least_period(const Window &w, int T, std::vector<int> &s)
{
    if (!least_starts(w, T, s)) return false;
    std::vector<int> other;
    if (!in_sequence(w, [&](const Edge &e) { return s[e.u] + e.w - e.lag * T == s[e.v]; }, other)) return true;
    return !least_starts(w, T - 1, other);
}

// ---- the candidate of the running best -----------------------------------------------------------------------------
// Leads, device orders after repair and peaks of one candidate from its index.  The blocks of one candidate follow one another, a few
// dependent instructions each: 256 blocks on 8 devices take a core 10 us, and took a wave of the GPU, a lane for every block
// type of every device, 38 (a call that scores 200,003 candidates of 16 devices and asks for the best 336 -> 307 us).
void decode_candidate(const tessel_problem *p, uint64_t idx, Detail &c)
{
    const KParams &kp = p->kp;
    const int D = kp.D, K = kp.K, NR = kp.NR;
    const bool sampled = kp.space == kSampledStrict || kp.space == kSampledRepair;
    uint8_t type[kMaxDW][kMaxLTW] = {}, order[kMaxDW][kMaxPos];
    for (int d = 0; d < D; d++)
        for (int y = 0; y < kp.ntd[d]; y++) type[d][y] = (uint8_t)((y < 4 ? kp.type_of[d] >> (8 * y) : kp.type_of_hi[d] >> (8 * (y - 4))) & 0xFFu);
    memset(&c, 0, sizeof c);
    c.index = idx;
    // producers and consumers
    uint64_t producers[kMaxKW] = {}, consumers[kMaxKW] = {};
    for (size_t e = 0; e < p->dep_src.size(); e++) {
        producers[p->dep_dst[e]] |= 1ull << p->dep_src[e];
        consumers[p->dep_src[e]] |= 1ull << p->dep_dst[e];
    }
    // ---- orders as drawn or unranked
    uint32_t ka = 0, kb = 0;
    if (sampled) ka = stream_keys(kp.seed, idx, kb);
    uint64_t rest = idx;
    for (int d = 0; d < D; d++) {
        const int types = kp.ntd[d], n = types * NR;
        if (sampled) {
            int left[kMaxLTW];
            for (int y = 0; y < types; y++) left[y] = NR;
            uint32_t word = 0;
            for (int pos = 0; pos < n; pos++) {
                const uint32_t j = kDrawOrdBase + 32u * (uint32_t)d + (uint32_t)pos;
                if ((pos & 1) == 0) word = stream_word(ka, kb, j >> 1);
                int digit = (int)((((word >> (16u * (j & 1u))) & 0xFFFFu) * (uint32_t)(n - pos)) >> 16), y = 0;
                while (digit >= left[y]) digit -= left[y++];
                left[y]--;
                order[d][pos] = (uint8_t)y;
            }
        } else if (kp.space == kCanonical) {
            const uint32_t B = (uint32_t)NR + 1;
            uint64_t r = rest % kp.cdev[d];
            rest /= kp.cdev[d];
            uint32_t left[kMaxLT];
            for (int y = 0; y < kMaxLT; y++) left[y] = y < types ? (uint32_t)NR : 0u;
            for (int pos = 0; pos < n; pos++)
                for (int y = 0; y < types; y++) {
                    if (left[y] == 0) continue;
                    left[y]--;
                    const uint64_t w = p->wtab[((left[0] * B + left[1]) * B + left[2]) * B + left[3]];
                    if (r < w) { order[d][pos] = (uint8_t)y; break; }
                    r -= w;
                    left[y]++;
                }
        } else {
            uint32_t r = (uint32_t)(rest % kp.cdev[d]);
            rest /= kp.cdev[d];
            uint64_t list = kp.init_list[d];
            bool seen[kMaxLT] = {};
            for (int pos = 0; pos < n; pos++) {
                const uint32_t f = kp.fact[n - 1 - pos], digit = r / f;
                r -= digit * f;
                const uint32_t code = (uint32_t)(list >> (5u * digit)) & 31u, y = code >> 3;
                const uint64_t low = list & ((1ull << (5u * digit)) - 1ull);
                list = low | (((list >> (5u * digit)) >> 5) << (5u * digit));
                order[d][pos] = (uint8_t)y;
                if (!seen[y]) { c.leads[type[d][y]] = (int)(code & 7u); seen[y] = true; }       // (one lead per type: the candidate is feasible)
            }
        }
    }
    // ---- leads
    if (kp.space == kCanonical)
        for (int g = 0; g < K; g++) c.leads[g] = p->leadtab[rest * (uint64_t)K + (uint64_t)g];
    else if (sampled && kp.has_fixed)
        for (int g = 0; g < K; g++) c.leads[g] = kp.fixed[g];
    else if (sampled) {
        // the least solution of lead = min(N_R - 1, largest consumer's lead + step)
        uint8_t step[kMaxDeps];
        const int deps = (int)p->dep_src.size();
        for (int e = 0; e < deps; e++)
            step[e] = p->mask[p->dep_src[e]] != p->mask[p->dep_dst[e]] && stream_draw16(ka, kb, kDrawLeadBase + (uint32_t)e) < kp.step_q16;
        for (bool grew = true; grew;) {
            grew = false;
            for (int e = deps - 1; e >= 0; e--) {
                const int v = std::min(NR - 1, c.leads[p->dep_dst[e]] + step[e]);
                if (v > c.leads[p->dep_src[e]]) { c.leads[p->dep_src[e]] = v; grew = true; }
            }
        }
    }
    // ---- blocks in an executable sequence: heads first, else (repair) the lowest device's earliest that may run
    uint32_t alive[kMaxDW], at[kMaxDW][kMaxLTW] = {};               // entries not yet placed, by device and by type
    uint64_t here[kMaxDW] = {};                                     // the types of a device
    int mem[kMaxDW], mu[kMaxKW], lists[kMaxKW] = {};                // memory now; next micro-batch; devices whose list the type heads
    uint64_t may = 0, heads = 0;                                    // types that may run; that head all their devices
    uint8_t home[kMaxKW] = {}, symbol[kMaxKW] = {};                 // lowest device and symbol there
    auto look = [&](int g) {
        bool ok = mu[g] < c.leads[g] + NR;
        for (uint64_t a = producers[g]; ok && a; a &= a - 1) ok = mu[__builtin_ctzll(a)] > mu[g];
        may = (may & ~(1ull << g)) | (uint64_t)ok << g;
    };
    auto new_head = [&](int d) {
        if (!alive[d]) return;
        const int g = type[d][order[d][__builtin_ctz(alive[d])]];
        if (++lists[g] == __builtin_popcount(p->mask[g])) heads |= 1ull << g;
    };
    for (int g = 0; g < K; g++) mu[g] = c.leads[g];
    for (int g = 0; g < K; g++) look(g);
    for (int d = D - 1; d >= 0; d--) {
        const int n = kp.ntd[d] * NR;
        alive[d] = n >= 32 ? 0xFFFFFFFFu : (1u << n) - 1u;
        mem[d] = 0;
        c.peak[d] = INT_MIN;
        for (int pos = 0; pos < n; pos++) at[d][order[d][pos]] |= 1u << pos;
        for (int y = 0; y < kp.ntd[d]; y++) {
            const int g = type[d][y];
            here[d] |= 1ull << g; home[g] = (uint8_t)d; symbol[g] = (uint8_t)y;
            mem[d] += kp.m_of[d][y] * c.leads[g];
        }
        new_head(d);
    }
    // takes the earliest entry of type g out of device d's list
    auto take = [&](int g, int d, int y) {
        const uint32_t first = alive[d] & (0u - alive[d]), bit = at[d][y] & (0u - at[d][y]);
        at[d][y] ^= bit;
        alive[d] ^= bit;
        if (bit == first) { lists[g]--; heads &= ~(1ull << g); new_head(d); }
        mem[d] += kp.m_of[d][y];
        c.peak[d] = std::max(c.peak[d], mem[d]);
        c.orders[d][c.order_len[d]++] = (uint8_t)g;
    };
    auto place = [&](int g) {
        take(g, home[g], symbol[g]);
        for (uint32_t on = p->mask[g] & (p->mask[g] - 1); on; on &= on - 1) {
            const int d = __builtin_ctz(on);
            int y = 0;
            while (type[d][y] != g) y++;
            take(g, d, y);
        }
        mu[g]++;
        look(g);
        for (uint64_t s = consumers[g]; s; s &= s - 1) look(__builtin_ctzll(s));
    };
    c.status = kOk;
    for (int placed = 0; placed < kp.total; placed++) {
        if (const uint64_t now = may & heads) { place(__builtin_ctzll(now)); continue; }
        int d = 0;
        if (kp.space == kSampledRepair) while (d < D && !(here[d] & may)) d++;
        if (kp.space != kSampledRepair || d == D) { c.status = kDeadlock; break; }
        uint32_t can = 0;
        for (int y = 0; y < kp.ntd[d]; y++) can |= may >> type[d][y] & 1 ? at[d][y] : 0u;
        place(type[d][order[d][__builtin_ctz(can)]]);
    }
    for (int d = 0; d < D; d++) {
        if (c.peak[d] == INT_MIN) c.peak[d] = 0;                    // a device without blocks
        if (c.status == kOk && c.peak[d] > kp.M) c.status = kMem;
    }
}

// p->starts and p->period_right of the running best just read, and of its window if it has one
void check_period(tessel_problem *p, bool executable, const Window &w, const std::vector<int> &rank)
{
    std::vector<int> s;
    p->starts.assign((size_t)p->kp.K * p->kp.NR, 0);
    p->period_right = executable && is_least_period(w, p->result.period, s);
    if (p->period_right)
        for (size_t k = 0; k < p->starts.size(); k++) p->starts[k] = s[rank[k]];
}

void check_period(tessel_problem *p)
{
    Window w;
    std::vector<int> rank;
    const bool executable = p->detail.status == kOk && make_window(p, p->detail, w, rank);
    check_period(p, executable, w, rank);
}

// The two counters of a record that scoring this candidate alone leaves behind: blocks placed, and the window sweeps of the fast kernel
// (period_fast).  One sweep: the end times of all blocks of one window after those of the window before, 0 before the first.
// The values whose growths tell the period: every device's last end, and for every chain and micro-batch on its way through
// it at the window's end the last end on that micro-batch.
void count_alone(const tessel_problem *p, const Window &w, const std::vector<int> &rank, DevResult &record)
{
    const KParams &kp = p->kp;
    const int NR = kp.NR;
    if (!kp.fast_ok || p->force_general) return;             // (the other kernels count neither)
    record.n_blocks = (uint64_t)kp.total;
    std::vector<int> values;
    for (int d = 0; d < kp.D; d++)
        if (const int n = p->detail.order_len[d]) values.push_back(rank[(int)p->detail.orders[d][n - 1] * NR + NR - 1]);
    for (int head = 0; head < kp.K; head++) {
        if (kp.pred[head] >= 0) continue;
        for (int m = 0; m < p->detail.leads[head]; m++) {
            int g = head;                                    // the last type of the chain that has handled micro-batch m + N_R
            while (kp.succ[g] >= 0 && p->detail.leads[kp.succ[g]] > m) g = kp.succ[g];
            values.push_back(rank[g * NR + m + NR - p->detail.leads[g]]);
        }
    }
    std::vector<int> end, before, grown(values.size()), was;
    // sweeps until the period shows, at most `tries`; `shown`: whether it did
    auto sweeps = [&](int tries, bool settle, bool &shown) -> int {
        end.assign(w.blocks, 0);
        int top_before = 0;
        for (int j = 0; j < tries; j++) {
            before = end;
            std::fill(end.begin(), end.end(), 0);
            for (const Edge &e : w.edges) if (e.lag) end[e.v] = std::max(end[e.v], before[e.u]);       // (start times so far)
            for (int u = 0; u < w.blocks; u++) {
                end[u] += w.edges[w.from[u]].w;
                for (int e = w.from[u]; e < w.from[u + 1]; e++)
                    if (!w.edges[e].lag) end[w.edges[e].v] = std::max(end[w.edges[e].v], end[u]);
            }
            for (size_t v = 0; v < values.size(); v++) grown[v] = end[values[v]] - before[values[v]];
            const int top = *std::max_element(grown.begin(), grown.end());
            shown = *std::min_element(grown.begin(), grown.end()) == top;
            if (settle && j > 0 && top == top_before) {
                bool held = true;
                for (size_t v = 0; v < values.size(); v++) held = held && (was[v] != top || grown[v] == top);
                shown = shown || held;
            }
            if (shown) return j + 1;
            top_before = top; was = grown;
        }
        return tries;
    };
    bool shown = false;
    record.n_sweeps = (uint64_t)sweeps(kp.eigen_tries, false, shown);
    if (!shown) {
        record.n_sweeps += (uint64_t)sweeps(kp.retry_tries, true, shown);
        record.n_retried = 1;
        record.n_deferred = shown ? 0 : 1;
    }
}

}  // namespace

// ---- mail: small results straight from a kernel into pinned host memory ---------------------------------------------
// A copy of 100 bytes to host memory through the runtime and the wait for it take 18 us, as long as scoring a thousand
// candidates; a kernel's own stores and a look at the last of them take 3 after the kernel's launch.  A few boxes serve all handles, threads
// and GPUs, one for the time of a call each; a call that finds none (or no pinned memory) copies as before.  The
// memory is allocated with the first call that could use it and freed when the process ends.
namespace {
constexpr int kMailboxes = 16;
std::mutex g_mail_mutex;
DevMail *g_mail = nullptr;
uint32_t g_mail_used = 0, g_mail_told = 0;

void free_mail()
{
    std::lock_guard<std::mutex> lock(g_mail_mutex);
    if (g_mail && g_mail_used == 0) (void)hipHostFree(g_mail);
    g_mail = nullptr;
    g_mail_used = ~0u;
}

class Mailbox {
public:
    DevMail *box = nullptr;
    uint32_t told = 0;
    explicit Mailbox(bool use)
    {
        if (!use) return;
        std::lock_guard<std::mutex> lock(g_mail_mutex);
        if (!g_mail && g_mail_used == 0) {
            void *mem = nullptr;
            if (hipHostMalloc(&mem, kMailboxes * sizeof(DevMail), hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
                (void)hipGetLastError();
                return;
            }
            g_mail = (DevMail *)mem;
            for (int k = 0; k < kMailboxes; k++) g_mail[k].told = 0;
            std::atexit(free_mail);
        }
        const uint32_t left = ~g_mail_used & ((1u << kMailboxes) - 1u);
        if (!g_mail || !left) return;
        at = __builtin_ctz(left);
        g_mail_used |= 1u << at;
        if (++g_mail_told == 0) g_mail_told = 1;
        told = g_mail_told;
        box = g_mail + at;
    }
    ~Mailbox()
    {
        if (!box || lost) return;
        std::lock_guard<std::mutex> lock(g_mail_mutex);
        g_mail_used &= ~(1u << at);
    }
    Mailbox(const Mailbox &) = delete;
    Mailbox &operator=(const Mailbox &) = delete;
    // `launched`: the status of the launch that sends the mail.  Waits until the mail is there: at first by looking at it, then by
    // waiting for the stream, which also finds out about a kernel that failed.  A box whose launch or kernel failed may still
    // be written to, and is not used again.
    int wait(int launched, hipStream_t st)
    {
        lost = true;
        if (launched) return launched;
        const int rc = arrived(st);
        lost = rc != 0;
        return rc;
    }
private:
    int at = 0;
    bool lost = false;
    int arrived(hipStream_t st) const
    {
        const auto start = std::chrono::steady_clock::now();
        for (int k = 1;; k++) {
            if (__atomic_load_n(&box->told, __ATOMIC_ACQUIRE) == told) return 0;
            if (k % 64 == 0 && std::chrono::steady_clock::now() - start > std::chrono::microseconds(200)) break;
            __builtin_ia32_pause();
        }
        const hipError_t e = hipStreamSynchronize(st);
        if (e != hipSuccess) return (int)e;
        return __atomic_load_n(&box->told, __ATOMIC_ACQUIRE) == told ? 0 : (int)hipErrorUnknown;
    }
};
}  // namespace

// The running best as it is on the device, into p->result and p->detail.  The record is read on every call: scoring
// launches that the caller captured in a graph change it when they are replayed, without a call of this library.  It names its
// candidate by the index, from which the host decodes it unless it did before.
static int read_back(tessel_problem *p)
{
    DevResult now;
    Mailbox mail(p->mail);
    if (mail.box) {
        const int le = mail.wait(launch_tell(p->ws, kWsResultOff, sizeof now, mail.box, mail.told, p->stream), p->stream);
        if (le) return hip_fail(p, le);
        memcpy(&now, mail.box->words, sizeof now);
    } else {
        hipError_t e = hipMemcpyAsync(&now, (char *)p->ws + kWsResultOff, sizeof now, hipMemcpyDeviceToHost, p->stream);
        if (e != hipSuccess) return hip_fail(p, (int)e);
        e = hipStreamSynchronize(p->stream);
        if (e != hipSuccess) return hip_fail(p, (int)e);
    }
    const bool known = now.period == p->result.period && now.index == p->result.index;
    p->result = now;
    if (now.period == INT_MAX || known) return TESSEL_OK;
    decode_candidate(p, now.index, p->detail);
    check_period(p);
    return TESSEL_OK;
}

static int fetch_best(tessel_problem *p)
{
    if (!p->ws || !p->ws_ready) { memset(&p->result, 0, sizeof p->result); p->result.period = INT_MAX; return TESSEL_OK; }
    if (!owns_workspace(p)) return TESSEL_E_WORKSPACE;       // another handle has bound the buffer since: the running best is gone
    int rc = read_back(p);
    if (rc) return rc;
    if (p->result.overflow && !p->safe_pieces) {
        // some launch left more candidates unfinished than its list holds, so the running best is incomplete:
        // score every range again, from now on in pieces small enough for the lists
        p->safe_pieces = true;
        p->best_dirty = true;
        int le = launch_reset(p->ws, p->stream);
        if (le) return hip_fail(p, le);
        for (const auto &r : p->ranges) {
            le = launch_eval(p->kp, r.first, r.second, p->ws, p->num_cus, p->max_blocks, p->stream, kSafePerLaunch);
            if (le) return hip_fail(p, le);
        }
        rc = read_back(p);
        if (rc) return rc;
    }
    if (p->result.period != INT_MAX) p->best_dirty = false;
    return TESSEL_OK;
}

extern "C" int tessel_best(tessel_problem *p, tessel_result *out)
{
    if (!p || !out) return TESSEL_E_INVALID_ARG;
    int rc = fetch_best(p);
    if (rc) return rc;
    memset(out, 0, sizeof *out);
    out->lower_bound = p->kp.LB;
    out->n_evaluated = p->result.n_evaluated;
    out->n_feasible = p->result.n_status[kOk];
    for (int s = 1; s < kNumStatus; s++) out->n_reject[s] = p->result.n_status[s];
    out->n_window_sweeps = p->result.n_sweeps;
    out->n_blocks_placed = p->result.n_blocks;
    if (p->result.overflow) return TESSEL_E_WORKSPACE;       // more candidates deferred than the list holds
    if (p->result.period == INT_MAX) { out->period = -1; return TESSEL_E_NO_FEASIBLE; }
    out->period = p->result.period;
    out->index = p->result.index;
    out->peak_max = INT_MIN;
    for (int d = 0; d < p->kp.D; d++) { out->peak_mem[d] = p->detail.peak[d]; out->peak_max = std::max(out->peak_max, p->detail.peak[d]); }
    if (!p->period_right) return TESSEL_E_HIP;               // the decoded candidate has another period: never expected
    return TESSEL_OK;
}

extern "C" int tessel_best_candidate(tessel_problem *p, int32_t *leads, int32_t *order_len, int32_t *orders, int32_t *starts)
{
    if (!p) return TESSEL_E_INVALID_ARG;
    int rc = fetch_best(p);
    if (rc) return rc;
    if (p->result.period == INT_MAX) return TESSEL_E_NO_FEASIBLE;
    const Detail &c = p->detail;
    if (leads) for (int i = 0; i < p->kp.K; i++) leads[i] = c.leads[i];
    if (order_len) for (int d = 0; d < p->kp.D; d++) order_len[d] = c.order_len[d];
    if (orders) for (int d = 0; d < p->kp.D; d++) for (int k = 0; k < kMaxPos; k++) orders[d * kMaxPos + k] = k < c.order_len[d] ? c.orders[d][k] : -1;
    if (starts) {
        if (!p->period_right) return TESSEL_E_HIP;           // no start times at that period: never expected
        std::copy(p->starts.begin(), p->starts.end(), starts);
    }
    return TESSEL_OK;
}

// Sec. IV-C.  Warm-up = blocks (i, mu) with mu < lead_i, steady = R windows, cool-down = the rest
// (Eq. 5-6 for every micro-batch the windows do not cover).  Warm-up and cool-down are ordered by a
// serial greedy list schedule: of the blocks of the phase that are ready (producers scheduled) and
// fit the cap on each device they occupy, append the one with the smallest (earliest start,
// micro-batch, type).  A block starts at the maximum of its devices' free times and its producers'
// ends, which is also the earliest start for the final per-device orders.
// Completion candidate `ordinal` with jitter amplitude J around R copies of the best window; ordinal 0 or
// J = 0: the plain greedy schedule.  Per phase every type offers its lowest unscheduled micro-batch.
static int complete_with(tessel_problem *p, tessel_schedule *out, uint64_t ordinal, int J)
{
    const Detail &c = p->detail;
    const int N = out->num_microbatches, K = p->kp.K, D = p->kp.D, NR = p->kp.NR, M = p->kp.M;
    int maxlead = 0;
    for (int i = 0; i < K; i++) maxlead = std::max(maxlead, c.leads[i]);
    const int R = N >= 1 ? (N - maxlead) / NR : 0;
    if (R < 1 || out->capacity < K * N) return TESSEL_E_RANGE;
    std::vector<int> finish(K * N, -1), next(K, 0);
    std::vector<int> dev_free(D, 0), dev_mem(D, 0);
    for (int d = 0; d < D; d++) out->dev_len[d] = 0;
    std::vector<std::vector<int>> producers(K);
    for (size_t e = 0; e < p->dep_src.size(); e++) producers[p->dep_dst[e]].push_back(p->dep_src[e]);
    uint32_t kb = 0;
    const uint32_t ka = stream_keys(p->kp.seed + kCompletionKey, ordinal, kb);
    const bool noisy = ordinal != 0 && J > 0;

    auto earliest = [&](int i, int mu, int &est) -> bool {      // false if a producer is not scheduled yet
        est = 0;
        for (int a : producers[i]) {
            if (next[a] <= mu) return false;
            est = std::max(est, finish[a * N + mu]);
        }
        for (int d = 0; d < D; d++) if (p->mask[i] >> d & 1u) est = std::max(est, dev_free[d]);
        return true;
    };
    auto commit = [&](int i, int mu, int est) {
        out->start[i * N + mu] = est;
        finish[i * N + mu] = est + p->t[i];
        next[i] = mu + 1;
        for (int d = 0; d < D; d++) if (p->mask[i] >> d & 1u) {
            dev_free[d] = est + p->t[i];
            dev_mem[d] += p->m[i];
            out->dev_order[(size_t)d * out->capacity + out->dev_len[d]++] = i * N + mu;
        }
    };
    auto greedy_phase = [&](bool warmup) -> int {
        for (;;) {
            int pick = -1, pick_mu = 0, pick_est = 0, pick_key = 0;
            bool left = false;
            for (int i = 0; i < K; i++) {
                const int hi = warmup ? c.leads[i] : N, mu = next[i];
                if (mu >= hi) continue;
                left = true;
                int est;
                if (!earliest(i, mu, est)) continue;
                bool fits = true;
                if (p->m[i] > 0)
                    for (int d = 0; d < D; d++) if ((p->mask[i] >> d & 1u) && dev_mem[d] + p->m[i] > M) fits = false;
                if (!fits) continue;
                const int key = est + (noisy ? (int)((stream_draw16(ka, kb, (uint32_t)(i * N + mu)) * (uint32_t)(J + 1)) >> 16) : 0);
                if (pick < 0 || key < pick_key || (key == pick_key && mu < pick_mu)) { pick = i; pick_mu = mu; pick_est = est; pick_key = key; }
            }
            if (!left) return TESSEL_OK;
            if (pick < 0) return TESSEL_E_NO_SCHEDULE;
            commit(pick, pick_mu, pick_est);
        }
    };

    int rc = greedy_phase(true);
    if (rc) return rc;
    for (int k = 0; k < R; k++) {
        // replay the window in any executable sequence of the decoded per-device orders
        std::vector<int> pos(D, 0);
        int left = K * NR;
        while (left > 0) {
            bool moved = false;
            for (int d = 0; d < D; d++) {
                if (pos[d] >= c.order_len[d]) continue;
                int i = c.orders[d][pos[d]], mu = next[i], est;
                bool heads = true;
                for (int dd = 0; dd < D; dd++)
                    if ((p->mask[i] >> dd & 1u) && (pos[dd] >= c.order_len[dd] || c.orders[dd][pos[dd]] != i)) heads = false;
                if (!heads || !earliest(i, mu, est)) continue;
                commit(i, mu, est);
                for (int dd = 0; dd < D; dd++) if (p->mask[i] >> dd & 1u) pos[dd]++;
                left--; moved = true;
            }
            if (!moved) return TESSEL_E_NO_SCHEDULE;
        }
    }
    rc = greedy_phase(false);
    if (rc) return rc;
    out->makespan = *std::max_element(finish.begin(), finish.end());
    out->period = p->result.period;
    out->num_windows = R;
    return TESSEL_OK;
}

extern "C" int tessel_complete_schedule(tessel_problem *p, tessel_schedule *out)
{
    if (!p || !out || !out->start || !out->dev_order || !out->dev_len) return TESSEL_E_INVALID_ARG;
    int rc = fetch_best(p);
    if (rc) return rc;
    if (p->result.period == INT_MAX) return TESSEL_E_NO_FEASIBLE;
    return complete_with(p, out, 0, 0);
}

// ---- searched completion: many perturbed greedy completions scored on the GPU -----------------------
// uploads what the kernel needs of the problem and of the best candidate (once per best candidate, N, J)
// The R replayed windows as a (max, +) matrix (CompMatrix).  A dry run of the replay finds the state slots read before they are written (the
// inputs) and the slots written (the outputs).  A run with every slot as a row of the longest paths from the inputs, an input's own 0 and
// the others "no path", gives the matrix.  (A run an input, over a list of the blocks of all windows: the first call for 16
// stages on 8 devices and 1,000 micro-batches 603 to 1,123 us, 246 so.)
static void window_matrix(const CompParams &cp, CompMatrix &cm)
{
    memset(&cm, 0, sizeof cm);
    const int TR = cp.tok_ring, tmask = TR - 1, oFree = cp.npaths * TR, nslot = oFree + cp.D;      // rings first, then the devices
    // a block of the window: its devices, the rings of its producers and its own (-1: none)
    struct Block { int t, mu, dev0, dev1, from0, from1, to; };
    std::vector<Block> blocks((size_t)cp.nseq);
    std::vector<int> devs, from;
    for (int s = 0; s < cp.nseq; s++) {
        const int i = cp.seq[s];
        Block &b = blocks[(size_t)s];
        b.t = cp.t[i]; b.mu = (int)cp.lead[i] + (int)cp.occ[s]; b.to = cp.path[i] != 0xFF ? (int)cp.path[i] * TR : -1;
        b.dev0 = (int)devs.size(); b.from0 = (int)from.size();
        for (unsigned on = cp.mask[i]; on; on &= on - 1) devs.push_back(oFree + __builtin_ctz(on));
        if (cp.dag) for (uint32_t rest = cp.predmask[i]; rest; rest &= rest - 1) from.push_back((int)cp.path[__builtin_ctz(rest)] * TR);
        else if (cp.pred[i] >= 0) from.push_back(b.to);
        b.dev1 = (int)devs.size(); b.from1 = (int)from.size();
    }
    std::vector<int> state(nslot, 0);                       // 0 untouched, 1 read first, 2 written first; then: written at all
    std::vector<char> written(nslot, 0);
    for (int k = 0; k < std::min(cp.R, TR); k++)            // (after TR windows the same entries of the rings again)
        for (const Block &b : blocks) {
            const int at = (b.mu + cp.NR * k) & tmask;
            for (int d = b.dev0; d < b.dev1; d++) { if (!state[devs[d]]) state[devs[d]] = 1; written[devs[d]] = 1; }
            for (int f = b.from0; f < b.from1; f++) if (!state[from[f] + at]) state[from[f] + at] = 1;
            if (b.to >= 0) { if (!state[b.to + at]) state[b.to + at] = 2; written[b.to + at] = 1; }
        }
    std::vector<int> in, out;
    for (int v = 0; v < nslot; v++) { if (state[v] == 1) in.push_back(v); if (written[v]) out.push_back(v); }
    if (in.empty() || (int)in.size() > kMatIn || (int)out.size() > kMatOut) return;
    struct Row { int32_t x[kMatIn]; };
    Row none;
    for (int j = 0; j < kMatIn; j++) none.x[j] = -(1 << 28);           // (times stay below 2^16)
    std::vector<Row> rows(nslot, none);
    for (size_t j = 0; j < in.size(); j++) rows[in[j]].x[j] = 0;
    for (int k = 0; k < cp.R; k++)
        for (const Block &b : blocks) {
            const int at = (b.mu + cp.NR * k) & tmask;
            Row end = rows[devs[b.dev0]];
            auto after = [&](const Row &r) { for (int j = 0; j < kMatIn; j++) end.x[j] = std::max(end.x[j], r.x[j]); };
            for (int d = b.dev0 + 1; d < b.dev1; d++) after(rows[devs[d]]);
            for (int f = b.from0; f < b.from1; f++) after(rows[from[f] + at]);
            for (int j = 0; j < kMatIn; j++) end.x[j] += b.t;
            for (int d = b.dev0; d < b.dev1; d++) rows[devs[d]] = end;
            if (b.to >= 0) rows[b.to + at] = end;
        }
    for (int o = 0; o < kMatOut; o++) for (int j = 0; j < kMatIn; j++) cm.a[o][j] = kNoPath;
    for (size_t o = 0; o < out.size(); o++) {
        bool any = false;                                   // every output must depend on some input
        for (size_t j = 0; j < in.size(); j++) {
            const int32_t path = rows[out[o]].x[j];
            if (path >= 0) { cm.a[o][j] = path; any = true; }
        }
        if (!any) return;
    }
    for (size_t j = 0; j < in.size(); j++) cm.in_slot[j] = (uint32_t)in[j];
    for (size_t o = 0; o < out.size(); o++) cm.out_slot[o] = (uint32_t)out[o];
    cm.nin = (int32_t)in.size(); cm.nout = (int32_t)out.size();
}

static int bind_completion(tessel_problem *p, int N, int J)
{
    if (p->ws && p->ws_ready && !owns_workspace(p)) return TESSEL_E_WORKSPACE;      // the buffer is another handle's by now
    // (problems beyond the limits of the fast kernel keep their types, devices and micro-batches in more bits than the
    // completion kernel's tables hold; their greedy completion needs no kernel)
    if (p->kp.D > kMaxD || p->kp.K > kMaxK || p->kp.many || p->kp.NR > kMaxNR) return TESSEL_E_UNSUPPORTED;
    if (p->comp_ready && !p->best_dirty && p->comp_index == p->result.index && p->result.period != INT_MAX && p->comp.N == N &&
        p->comp.J == J)
        return TESSEL_OK;                                   // nothing new since the best was fetched: no wait
    int rc = fetch_best(p);
    if (rc) return rc;
    if (p->result.period == INT_MAX) return TESSEL_E_NO_FEASIBLE;
    if (p->comp_ready && p->comp_index == p->result.index && p->comp.N == N && p->comp.J == J) return TESSEL_OK;
    const Detail &c = p->detail;
    const int K = p->kp.K, D = p->kp.D, NR = p->kp.NR;
    if (N < 1 || J < 0 || J > 65535) return TESSEL_E_INVALID_ARG;
    int maxlead = 0;
    for (int i = 0; i < K; i++) maxlead = std::max(maxlead, c.leads[i]);
    const int R = (N - maxlead) / NR;
    if (R < 1) return TESSEL_E_RANGE;
    CompParams &cp = p->comp;
    memset(&cp, 0, sizeof cp);
    cp.D = D; cp.K = K; cp.NR = NR; cp.M = p->kp.M; cp.N = N; cp.J = J; cp.R = R; cp.nseq = K * NR;
    { const uint64_t seed = p->kp.seed + kCompletionKey; cp.seed_lo = (uint32_t)seed; cp.seed_hi = (uint32_t)(seed >> 32); }
    int npaths = 0;
    std::vector<std::vector<int>> producers(K);
    for (size_t e = 0; e < p->dep_src.size(); e++) producers[p->dep_dst[e]].push_back(p->dep_src[e]);
    for (int i = 0; i < K; i++) {
        if (p->m[i] < -128 || p->m[i] > 127) return TESSEL_E_UNSUPPORTED;
        cp.t[i] = p->t[i]; cp.m[i] = (int8_t)p->m[i]; cp.mask[i] = (uint8_t)p->mask[i];
        cp.pred[i] = p->kp.dag ? (int8_t)-1 : p->kp.pred[i];
        cp.lead[i] = (uint8_t)c.leads[i];
    }
    if (p->kp.dag) {
        // any acyclic graph: every type somebody consumes keeps the end times of its own blocks
        cp.dag = 1;
        std::vector<char> consumed(K, 0);
        for (size_t e = 0; e < p->dep_src.size(); e++) { consumed[p->dep_src[e]] = 1; cp.predmask[p->dep_dst[e]] |= 1u << p->dep_src[e]; }
        for (int i = 0; i < K; i++) cp.path[i] = consumed[i] ? (uint8_t)npaths++ : (uint8_t)0xFF;
    } else
    for (int i = 0; i < K; i++) if (p->kp.pred[i] < 0) {                 // chains numbered by their first type
        for (int g = i; g >= 0; g = p->kp.succ[g]) cp.path[g] = (uint8_t)npaths;
        npaths++;
    }
    cp.npaths = npaths;
    {
        // Phases and windows follow one another for all types together, so two types are never further apart than
        // (largest - smallest lead) + NR micro-batches; a ring of the next power of two above that holds every
        // micro-batch still on its way through a chain
        int lo = c.leads[0], hi = c.leads[0];
        for (int i = 1; i < K; i++) { lo = std::min(lo, c.leads[i]); hi = std::max(hi, c.leads[i]); }
        int ring = 1;
        while (ring < hi - lo + NR + 1) ring *= 2;
        cp.tok_ring = ring;
    }
    // one executable sequence of the window (the device orders of the best candidate)
    {
        std::vector<int> pos(D, 0), occ(K, 0);
        int n = 0;
        while (n < K * NR) {
            bool moved = false;
            for (int d = 0; d < D; d++) {
                if (pos[d] >= c.order_len[d]) continue;
                const int i = c.orders[d][pos[d]];
                bool heads = true;
                for (int dd = 0; dd < D; dd++)
                    if ((p->mask[i] >> dd & 1u) && (pos[dd] >= c.order_len[dd] || c.orders[dd][pos[dd]] != i)) heads = false;
                // its producers' blocks of the same micro-batch must come first: in this window, or they ran in an earlier one
                bool fed = true;
                for (int a : producers[i]) if (c.leads[a] + occ[a] <= c.leads[i] + occ[i]) fed = false;
                if (!heads || !fed) continue;
                cp.seq[n] = (uint8_t)i; cp.occ[n] = (uint8_t)occ[i]; n++;
                occ[i]++;
                for (int dd = 0; dd < D; dd++) if (p->mask[i] >> dd & 1u) pos[dd]++;
                moved = true;
            }
            if (!moved) return TESSEL_E_NO_SCHEDULE;
        }
    }
    {
        // the kernel keeps times, memory and jitter in 16 bits
        long long total = 0;
        for (int i = 0; i < K; i++) total += (long long)p->t[i] * N;
        if (total + J > 65535 || std::abs(p->kp.M) > 30000 || N > 1023 || J > 63) return TESSEL_E_TOOBIG;
    }

    window_matrix(cp, p->comp_matrix);
    if (const char *env = getenv("TESSEL_REPLAY_BLOCKS")) {        // test knob: replay the windows block by block
        if (env[0] == '1') p->comp_matrix.nin = 0;
    }
    if (!completion_fits(cp, p->comp_matrix)) return TESSEL_E_TOOBIG;
    hipError_t e = hipMemcpyAsync((char *)p->ws + kWsCompParamsOff, &cp, sizeof cp, hipMemcpyHostToDevice, p->stream);
    if (e != hipSuccess) return hip_fail(p, (int)e);
    e = hipMemcpyAsync((char *)p->ws + kWsCompMatrixOff, &p->comp_matrix, sizeof(CompMatrix), hipMemcpyHostToDevice, p->stream);
    if (e != hipSuccess) return hip_fail(p, (int)e);
    int le = launch_completion_reset(p->ws, p->stream);
    if (le) return hip_fail(p, le);
    p->comp_ready = true; p->comp_index = p->result.index;
    return TESSEL_OK;
}

extern "C" int tessel_search_completions(tessel_problem *p, int32_t num_microbatches, int32_t jitter, uint64_t first,
                                         uint64_t count)
{
    if (!p) return TESSEL_E_INVALID_ARG;
    if (first + count < first) return TESSEL_E_RANGE;
    int rc = bind_completion(p, num_microbatches, jitter);
    if (rc) return rc;
    int e = launch_completions(p->comp, p->comp_matrix, first, count, nullptr, p->ws, p->num_cus, p->stream);
    return e < 0 ? TESSEL_E_TOOBIG : e ? hip_fail(p, e) : TESSEL_OK;
}

extern "C" int tessel_score_completions(tessel_problem *p, int32_t num_microbatches, int32_t jitter, uint64_t first,
                                        uint64_t count, int32_t *makespan_dev)
{
    if (!p || !makespan_dev) return TESSEL_E_INVALID_ARG;
    if (first + count < first) return TESSEL_E_RANGE;
    int rc = bind_completion(p, num_microbatches, jitter);
    if (rc) return rc;
    int e = launch_completions(p->comp, p->comp_matrix, first, count, makespan_dev, p->ws, p->num_cus, p->stream);
    return e < 0 ? TESSEL_E_TOOBIG : e ? hip_fail(p, e) : TESSEL_OK;
}

extern "C" int tessel_best_completion(tessel_problem *p, tessel_schedule *out, uint64_t *ordinal)
{
    if (!p || !out || !out->start || !out->dev_order || !out->dev_len) return TESSEL_E_INVALID_ARG;
    if (!p->comp_ready || !p->ws) return TESSEL_E_NO_FEASIBLE;
    if (!owns_workspace(p)) return TESSEL_E_WORKSPACE;
    if (out->num_microbatches != p->comp.N) return TESSEL_E_INVALID_ARG;
    DevCompletion best;
    {
        Mailbox mail(p->mail);
        if (mail.box) {
            const int le = mail.wait(launch_tell(p->ws, kWsCompletionOff, sizeof best, mail.box, mail.told, p->stream), p->stream);
            if (le) return hip_fail(p, le);
            memcpy(&best, mail.box->words, sizeof best);
        } else {
            hipError_t e = hipStreamSynchronize(p->stream);
            if (e == hipSuccess) e = hipMemcpy(&best, (char *)p->ws + kWsCompletionOff, sizeof best, hipMemcpyDeviceToHost);
            if (e != hipSuccess) return hip_fail(p, (int)e);
        }
    }
    if (best.makespan == INT_MAX) return TESSEL_E_NO_SCHEDULE;
    int rc = complete_with(p, out, best.ordinal, p->comp.J);
    if (rc) return rc;
    if (out->makespan != best.makespan) return TESSEL_E_HIP;        // host and kernel disagree: never expected
    if (ordinal) *ordinal = best.ordinal;
    return TESSEL_OK;
}

// ---- Sec. IV-D: global sequence of blocks and send/receive pairs -----------------------------------
extern "C" int tessel_instantiate(const tessel_problem *p, const tessel_schedule *sched, tessel_op *ops, int32_t capacity,
                                  int32_t *num_ops)
{
    if (!p || !sched || !sched->start || !num_ops || (capacity > 0 && !ops) || sched->num_microbatches < 1)
        return TESSEL_E_INVALID_ARG;
    const int K = p->kp.K, D = p->kp.D, N = sched->num_microbatches;
    const int ndeps = (int)p->dep_src.size();
    for (int x = 0; x < K * N; x++) if (sched->start[x] < 0) return TESSEL_E_INVALID_ARG;
    auto lowest = [](uint32_t mask) { int d = 0; while (!(mask >> d & 1u)) d++; return d; };
    // blocks by (start time, lowest device); two blocks of one device never start together (t >= 1)
    std::vector<int> seq(K * N);
    for (int x = 0; x < K * N; x++) seq[x] = x;
    std::stable_sort(seq.begin(), seq.end(), [&](int a, int b) {
        if (sched->start[a] != sched->start[b]) return sched->start[a] < sched->start[b];
        return lowest(p->mask[a / N]) < lowest(p->mask[b / N]);
    });
    std::vector<tessel_op> out;
    out.reserve((size_t)K * N * 2);
    for (size_t at = 0; at < seq.size();) {
        size_t end = at;
        while (end < seq.size() && sched->start[seq[end]] == sched->start[seq[at]]) end++;
        for (size_t k = at; k < end; k++)
            out.push_back({TESSEL_OP_BLOCK, seq[k], (int32_t)p->mask[seq[k] / N], sched->start[seq[k]], 0});
        for (size_t k = at; k < end; k++) {
            const int i = seq[k] / N, mu = seq[k] % N;
            for (int e = 0; e < ndeps; e++) {
                if (p->dep_src[e] != i) continue;
                const int j = p->dep_dst[e];
                const uint32_t need = p->mask[j] & ~p->mask[i];        // consumer devices without the tensor
                for (int v = 0; v < D; v++)
                    if (need >> v & 1u) out.push_back({TESSEL_OP_SENDRECV, seq[k], lowest(p->mask[i]), v, j * N + mu});
            }
        }
        at = end;
    }
    *num_ops = (int32_t)out.size();
    if ((size_t)capacity < out.size()) return TESSEL_E_RANGE;
    std::copy(out.begin(), out.end(), ops);
    return TESSEL_OK;
}

// ---- Alg. 1: the loop over window sizes around the scoring kernels -------------------------

// CalMaxInflight of Alg. 1 (the paper gives no formula): one micro-batch alone, blocks in topological
// order with the smallest type id first, holds at most hold_d on device d; floor(M / hold_d) of them fit.
static int max_inflight(const tessel_problem_desc *desc, int unbounded)
{
    const int K = desc->num_block_types;
    std::vector<int> indeg(K, 0), done(K, 0), topo;
    for (int e = 0; e < desc->num_deps; e++) indeg[desc->dep_dst[e]]++;
    for (;;) {
        int pick = -1;
        for (int i = 0; i < K; i++) if (!done[i] && indeg[i] == 0) { pick = i; break; }
        if (pick < 0) break;
        done[pick] = 1; topo.push_back(pick);
        for (int e = 0; e < desc->num_deps; e++) if (desc->dep_src[e] == pick) indeg[desc->dep_dst[e]]--;
    }
    int best = unbounded;
    for (int d = 0; d < desc->num_devices; d++) {
        int run = 0, hold = 0;
        for (int i : topo) if (desc->dev_mask[i] >> d & 1u) { run += desc->mem[i]; hold = std::max(hold, run); }
        if (hold > 0) best = std::min(best, desc->mem_cap / hold);
    }
    return best;
}

extern "C" int tessel_search_workspace_bytes(const tessel_problem_desc *desc, const tessel_search *in, size_t *bytes)
{
    if (!desc || !in || !bytes || in->max_nr < 1 || in->max_nr > TESSEL_MAX_NR) return TESSEL_E_INVALID_ARG;
    size_t need = 0;
    int limit = in->max_nr;
    for (int nr = 1; nr <= limit; nr++) {
        tessel_problem_desc d = *desc;
        d.nr = nr; d.fixed_leads = nullptr;
        tessel_problem *p = nullptr;
        int rc = tessel_problem_create(&d, &p);
        if (rc) return rc;
        if (nr == 1 && in->use_inflight_bound) limit = std::max(1, std::min(limit, max_inflight(desc, in->max_nr)));
        size_t b = 0;
        rc = tessel_workspace_bytes(p, &b);
        tessel_problem_destroy(p);
        if (rc) return rc;
        need = std::max(need, b);
    }
    *bytes = need;
    return TESSEL_OK;
}

extern "C" int tessel_search_run(const tessel_problem_desc *desc, tessel_search *io, void *workspace_dev,
                                 size_t workspace_bytes, void *hip_stream, tessel_problem **best_out)
{
    if (best_out) *best_out = nullptr;
    if (!desc || !io || io->max_nr < 1 || io->max_nr > TESSEL_MAX_NR) return TESSEL_E_INVALID_ARG;
    const uint64_t per_launch = io->launch_candidates ? io->launch_candidates : (uint64_t)1 << 24;
    io->inflights = 0; io->lower_bound = 0; io->nr_tried = 0; io->best_nr = 0; io->best_period = -1;
    io->early_exit = 0; io->best_index = 0;
    for (int n = 0; n <= TESSEL_MAX_NR; n++) { io->period_nr[n] = -1; io->index_nr[n] = 0; io->evaluated_nr[n] = 0; }

    int limit = io->max_nr;
    for (int nr = 1; nr <= limit && !io->early_exit; nr++) {
        tessel_problem_desc d = *desc;
        d.nr = nr; d.fixed_leads = nullptr;
        tessel_problem *p = nullptr;
        int rc = tessel_problem_create(&d, &p);
        if (rc) return rc;
        if (nr == 1) {
            io->lower_bound = p->kp.LB;
            io->inflights = max_inflight(desc, io->max_nr);
            if (io->use_inflight_bound) limit = std::min(limit, io->inflights);
            if (limit < 1) { tessel_problem_destroy(p); break; }
        }
        io->nr_tried = nr;
        const uint64_t n = std::min(p->count, io->max_candidates);
        tessel_result r;
        for (uint64_t first = 0; first < n && !io->early_exit; first += per_launch) {
            const uint64_t cnt = std::min(per_launch, n - first);
            rc = tessel_eval_candidates(p, first, cnt, workspace_dev, workspace_bytes, hip_stream);
            if (rc) { tessel_problem_destroy(p); return rc; }
            rc = tessel_best(p, &r);                                  // waits for the launch
            if (rc && rc != TESSEL_E_NO_FEASIBLE) { tessel_problem_destroy(p); return rc; }
            io->evaluated_nr[nr] = r.n_evaluated;
            if (rc == TESSEL_OK) {
                io->period_nr[nr] = r.period; io->index_nr[nr] = r.index;
                // launches ascend in index, so the running best is what a candidate-by-candidate scan
                // would hold after the first candidate that reaches the bound
                if (r.period == nr * io->lower_bound) io->early_exit = 1;
            }
        }
        if (io->period_nr[nr] >= 0 &&
            (io->best_period < 0 || (int64_t)io->period_nr[nr] * io->best_nr < (int64_t)io->best_period * nr)) {
            io->best_period = io->period_nr[nr]; io->best_nr = nr; io->best_index = io->index_nr[nr];
        }
        tessel_problem_destroy(p);
    }
    if (io->best_nr == 0) return TESSEL_E_NO_FEASIBLE;
    if (best_out) {
        tessel_problem_desc d = *desc;
        d.nr = io->best_nr; d.fixed_leads = nullptr;
        tessel_problem *p = nullptr;
        int rc = tessel_problem_create(&d, &p);
        if (rc) return rc;
        // (The incumbent as the only candidate scored.  Its period is checked like that of every record read back, while the copy is on its way.
        // Once this returns nothing is to come that would write the workspace, on whatever stream the caller uses it then.)
        DevResult best;
        memset(&best, 0, sizeof best);
        best.period = io->best_period; best.index = io->best_index; best.n_evaluated = 1; best.n_status[kOk] = 1;
        decode_candidate(p, best.index, p->detail);
        Window w;
        std::vector<int> rank;
        const bool executable = p->detail.status == kOk && make_window(p, p->detail, w, rank);
        if (executable) count_alone(p, w, rank, best);
        rc = bind_workspace(p, workspace_dev, workspace_bytes, (hipStream_t)hip_stream, 0, &best);
        if (rc) { tessel_problem_destroy(p); return rc; }
        p->stream = (hipStream_t)hip_stream;
        p->ranges.push_back({io->best_index, 1});
        p->result = best;
        check_period(p, executable, w, rank);
        // (asked again and again: hipStreamSynchronize took 5 us more)
        hipError_t e;
        while ((e = hipStreamQuery((hipStream_t)hip_stream)) == hipErrorNotReady) { }
        if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();       // (no later launch of this thread fails by it)
        if (e != hipSuccess || !p->period_right) { tessel_problem_destroy(p); return TESSEL_E_HIP; }      // (the latter never expected)
        *best_out = p;
    }
    return TESSEL_OK;
}

extern "C" int tessel_last_hip_error(const tessel_problem *p) { return p ? p->last_hip : 0; }
