// An image's tables and rows as the kernels lay them out in LDS (stage_tables and stage_rows in jpgd_kernels.h), made on the
// host from a parsed file.  Test code: the library never calls it.
#pragma once
#include <vector>

#include "../../include/jpgd.h"
#include "../../paper_2111_09219_amd/csrc/jpgd_lane.h"
#include "../../paper_2111_09219_amd/csrc/jpgd_lut.h"
#include "jpgd_plain.h"

namespace jpgd {

constexpr uint32_t kBase = 176, kRow0 = 48;  // bytes at which the tables and the rows start

struct Tables {
    std::vector<uint16_t> lut;    // build_lut, DC slots first
    std::vector<uint32_t> sync;   // the kernels' layout: synchronisation pass,
    std::vector<uint32_t> write;  // write pass
    uint32_t ndc = 0, nslots = 0;
    uint32_t words[6] = {0};      // sync_sub_words
};

// as stage_tables fills them, DC subtables in the order of their entries
template <bool WRITE>
bool lay_out(Tables& t, uint32_t base, std::vector<uint32_t>& out) {
    const uint32_t nac = t.nslots - t.ndc;
    std::vector<uint8_t> pairs(kPairBytes);
    uint32_t sub = t.ndc * kSyncDcBytes + nac * kSyncAcBytes, all = 0;
    for (uint32_t s = 0; s < t.nslots; ++s) all += t.words[s] = sync_sub_words(&t.lut[s * kLutEntries], s < t.ndc);
    out.assign(sub / 4 + all, 0xDEADBEEFu);
    for (uint32_t a = 0; a < nac; ++a) {
        const uint16_t* lut = &t.lut[(t.ndc + a) * kLutEntries];
        build_pairs(lut, pairs.data());
        for (uint32_t i = 0; i < (uint32_t)kLutL1; ++i)
            out[(t.ndc * kSyncDcBytes + a * kSyncAcBytes) / 4 + i] = sync_ac_entry<WRITE>(i, lut[i], pairs[i], base + sub);
        for (uint32_t k = 0; k < t.words[t.ndc + a]; ++k) out[sub / 4 + k] = pass_entry<WRITE>(lut[kLutL1 + k], false, 0u);
        sub += 4u * t.words[t.ndc + a];
    }
    for (uint32_t s = 0; s < t.ndc; ++s) {
        const uint16_t* lut = &t.lut[s * kLutEntries];
        for (uint32_t i = 0; i < 1u << kSyncDcK; ++i) {
            const uint32_t a = lut[2 * i], b = lut[2 * i + 1], n = sync_dc_sub(a, b);
            uint32_t& e = out[s * kSyncDcBytes / 4 + i];
            if (n == 0xFFFFFFFFu) { e = sync_dc_direct<WRITE>(a); continue; }
            e = sync_escape(n + 1u, base + sub);
            for (uint32_t j = 0; j < 2u << n; ++j, sub += 4)
                out.at(sub / 4) = sync_dc_sub_entry<WRITE>(a, b, n, j, lut + kLutL1);
        }
    }
    return sub / 4 == out.size();
}

// What a scan's decoders need to know: table slots in order of first use, as the library numbers them.
struct Layout {
    Tables t;
    uint32_t upm = 0, sched_dc = 0, sched_ac = 0, sched_comp = 0, walk = 0;
    SyncRow srows[8], wrows[8];  // synchronisation and write pass
    PlainUnit units[8];

    uint32_t component(uint32_t u) const { return (sched_comp >> (4u * u)) & 15u; }
    uint32_t sync_entry_at(uint32_t k) const { if (k < kBase || (k & 3u)) __builtin_trap(); return t.sync.at((k - kBase) / 4); }
    uint32_t write_entry_at(uint32_t k) const { if (k < kBase || (k & 3u)) __builtin_trap(); return t.write.at((k - kBase) / 4); }
    uint32_t unit_of_row(uint32_t k) const {
        if (k < kRow0 || (k - kRow0) % sizeof(SyncRow) || (k - kRow0) / sizeof(SyncRow) >= upm) __builtin_trap();
        return (k - kRow0) / (uint32_t)sizeof(SyncRow);
    }
    SyncRow sync_row_at(uint32_t k) const { return srows[unit_of_row(k)]; }
    SyncRow write_row_at(uint32_t k) const { return wrows[unit_of_row(k)]; }
};

inline int make_layout(const jpgd_info& in, Layout& y) {
    uint32_t ids[2][3], n[2] = {0, 0}, slot[2][3];
    for (uint32_t cls = 0; cls < 2; ++cls)
        for (uint32_t c = 0; c < in.ncomp; ++c) {
            const uint32_t id = cls ? in.ta[c] : in.td[c];
            uint32_t k = 0;
            while (k < n[cls] && ids[cls][k] != id) ++k;
            if (k == n[cls]) ids[cls][n[cls]++] = id;
            slot[cls][c] = k;
        }
    y.t.ndc = n[0];
    y.t.nslots = n[0] + n[1];
    y.t.lut.assign((size_t)y.t.nslots * kLutEntries, 0);
    for (uint32_t cls = 0; cls < 2; ++cls)
        for (uint32_t k = 0; k < n[cls]; ++k)
            if (!build_lut(in.dht_bits[cls][ids[cls][k]], in.dht_vals[cls][ids[cls][k]], cls == 0, &y.t.lut[(size_t)(cls * n[0] + k) * kLutEntries]))
                return JPGD_E_TABLE;
    if (!lay_out<false>(y.t, kBase, y.t.sync) || !lay_out<true>(y.t, kBase, y.t.write)) return JPGD_E_TABLE;
    uint32_t u = 0;
    for (uint32_t c = 0; c < in.ncomp; ++c)
        for (uint32_t k = 0, nu = in.ncomp == 3 && c == 0 ? (uint32_t)in.hsamp[0] * in.vsamp[0] : 1u; k < nu; ++k, ++u) {
            y.sched_dc |= slot[0][c] << (4 * u);
            y.sched_ac |= (n[0] + slot[1][c]) << (4 * u);
            y.sched_comp |= c << (4 * u);
        }
    y.upm = u;
    y.walk = walk_word(u, y.sched_dc, y.sched_ac);
    for (uint32_t k = 0; k < u; ++k) {
        const uint32_t next = k + 1 == u ? 0 : k + 1, dc = (y.sched_dc >> (4 * k)) & 15, ac = (y.sched_ac >> (4 * k)) & 15;
        y.units[k] = PlainUnit{dc * (uint32_t)kLutEntries, ac * (uint32_t)kLutEntries, y.component(k)};
        y.srows[k] = SyncRow{kBase + n[0] * kSyncDcBytes + (ac - n[0]) * kSyncAcBytes, kBase + ((y.sched_dc >> (4 * next)) & 15) * kSyncDcBytes,
                             1u << (15 * y.component(k)), kRow0 + next * (uint32_t)sizeof(SyncRow)};
        y.wrows[k] = y.srows[k];
        y.wrows[k].dcmul = y.component(k) != y.component(next) ? 1u : 0u;
    }
    return JPGD_OK;
}

}  // namespace jpgd
