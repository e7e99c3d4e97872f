// The walk of a whole wavefront through a single chain (coop_span_kinds in jpgd_kernels.h) with its 64 lanes run one after
// another: the same windows of 64 bits, one answer per lane and table, the same word S of position and index, the same sums.
// (The kernel asks for a window's answers one window ahead, and follows up the escapes of all lanes at the first one the
// chain meets; here each is followed up when the chain meets it, which gives the same entries.)  Test code: the library never
// calls it.
#pragma once
#include <stdlib.h>

#include "../../paper_2111_09219_amd/csrc/jpgd_lane.h"

namespace jpgd {

struct Walk {
    uint32_t unit_word[64], upm, dc[3], ac[3];
    bool three;
};
// tab: byte at which the tables begin
inline Walk make_walk(uint32_t walk, uint32_t sched_comp, uint32_t upm, uint32_t ndc, uint32_t tab) {
    Walk w;
    w.upm = upm;
    for (uint32_t u = 0; u < 64u; ++u) w.unit_word[u] = u < upm ? walk_unit(walk, sched_comp, upm, u) : 0u;
    for (uint32_t k = 0; k < 3u; ++k) { w.dc[k] = walk_dc(walk, k, tab); w.ac[k] = walk_ac(walk, k, ndc, tab); }
    w.three = (walk >> kWalkThree) & 1u;
    return w;
}

// p, u, z advanced until p >= limit; word(b): the stream word that starts at bit b, tab(k): entry at byte k.  `exact`: the
// three DC sums in full.
template <class Word, class Tab>
void walk_span(uint32_t& p, uint32_t& u, uint32_t& z, uint32_t& nb, int64_t& dc, int32_t exact[3], uint32_t limit, const Walk& w,
               Word word, Tab tab) {
    uint32_t ws = p & ~63u, S = (p - ws) | (z << 9), cur = w.unit_word[u], dc_a = 0u, dc_b = 0u;
    nb = 0u;
    exact[0] = exact[1] = exact[2] = 0;
    for (uint32_t left = (limit - ws) >> 6; left != 0u; --left, ws += 64u, S -= 64u) {
        uint32_t peek[64], d[3][64], a[3][64];
        for (uint32_t lane = 0; lane < 64u; ++lane) {
            const uint32_t b = ws + ((lane + 31u) >> 5) * 32u;   // of the second of the two words
            peek[lane] = funnel(lane ? word(b - 32u) : 0u, word(b), 0u - lane);
            for (uint32_t k = 0; k < 3u; ++k) {
                d[k][lane] = tab(w.dc[k] + ((peek[lane] >> (32u - kSyncDcK)) << 2));
                a[k][lane] = tab(w.ac[k] + ((peek[lane] >> (32u - kSyncAcK)) << 2));
            }
        }
        if ((S & 0x7Fu) >= 64u) abort();   // a chain enters a window inside it
        while (!(S & 0x40u)) {
            uint32_t kind = (cur >> kUwKind) & 3u;
            if (kind > (w.three ? 2u : 1u)) abort();
            if (S < 0x200u) {
                uint32_t r = d[kind][S];
                if (r >> 31) r = tab(sync_escape_at(r, peek[S]));
                const int32_t v = symbol_value(peek[S], r & 31u, (r >> 20) & 15u);
                const uint32_t comp = (cur >> kUwSecond) & 1u ? 2u : (cur >> kUwShift) & 31u ? 1u : 0u;
                exact[comp] += v;
                (comp == 2u ? dc_b : dc_a) += (uint32_t)v << ((cur >> kUwShift) & 31u);
                S += r & kSyncStep;
                if (S < 0x200u) abort();
                continue;
            }
            uint32_t e = a[kind][S & 63u];
            if (e & kSyncEsc) e = tab(sync_escape_at(e, peek[S & 63u]));
            S += e & kSyncStep;
            if (S & kSyncEsc) {
                ++nb;
                S &= 0x7Fu;
                cur = w.unit_word[cur & 15u];
            }
        }
    }
    p = limit + (S & 0x7Fu);
    z = S >> 9;
    const uint32_t next = cur & 15u;
    u = next == 0u ? w.upm - 1u : next - 1u;
    const int32_t s0 = (int32_t)(int16_t)(dc_a & 0xFFFFu), s1 = (int32_t)(dc_a - (uint32_t)s0) >> 16;
    dc = (int64_t)s0 + (int64_t)s1 * (1 << 15) + (int64_t)(int32_t)dc_b * (1 << 30);
}

}  // namespace jpgd
