// Host build of the kernels' lanes (sync_span, write_span and their _rst forms) and of the walk on tables laid out as the kernels
// lay them out in LDS, beside the plain lanes of jpgd_plain.h.  Test code: the library never calls it.
//
// Build: g++ -O2 -std=c++17 -shared -fPIC -o libjpgd_sync.so jpgd_sync.cpp ../../paper_2111_09219_amd/csrc/jpgd_parse.cpp
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <utility>
#include <vector>

#include "jpgd_tables.h"
#include "jpgd_walk.h"

using namespace jpgd;

namespace {

struct Scan {
    jpgd_info in;
    Layout y;
    std::vector<uint8_t> stream;
    std::vector<uint32_t> bmap;
    uint32_t nbits = 0;

    uint32_t word(uint32_t k) const { return k < stream.size() / 4 ? __builtin_bswap32(((const uint32_t*)stream.data())[k]) : 0u; }
    uint32_t peek(uint32_t p) const { return (uint32_t)(((((uint64_t)word(p >> 5) << 32) | word((p >> 5) + 1u)) << (p & 31u)) >> 32); }
};

struct Random {
    uint64_t r;
    explicit Random(uint32_t seed) : r(seed * 2654435761ull + 88172645463325252ull) {}
    uint32_t operator()(uint32_t n) { r ^= r << 13; r ^= r >> 7; r ^= r << 17; return (uint32_t)(r % n); }
};

int open_scan(const uint8_t* file, size_t len, Scan& S) {
    int rc = jpgd_parse(file, len, &S.in);
    if (rc || (rc = make_layout(S.in, S.y))) return rc;
    const jpgd_info& in = S.in;
    const uint8_t* p = file + in.scan_offset;
    S.bmap.assign(in.scan_bytes / 32 + 80, 0);
    for (size_t k = 0; k < in.scan_bytes; ++k) {
        if (p[k] == 0xFF && k + 1 < in.scan_bytes && p[k + 1] >= 0xD0 && p[k + 1] <= 0xD7) {
            S.bmap[S.stream.size() >> 5] |= 1u << (S.stream.size() & 31);
            ++k;
            continue;
        }
        S.stream.push_back(p[k]);
        if (p[k] == 0xFF) ++k;   // the stuffed zero
    }
    S.nbits = (uint32_t)S.stream.size() * 8;
    S.stream.resize(S.stream.size() + 1024, 0);
    return JPGD_OK;
}

}  // namespace

// `tries` random states, each decoded over `spans` subsequences of L bits by both: mismatches in state, unit count, DC sums or
// "an interval began".  org: added to the positions the lanes of sync_span see (a multiple of 32).  *compared: spans compared.
extern "C" int sync_vs_plain(const uint8_t* file, size_t len, uint32_t L, uint32_t tries, uint32_t spans, uint32_t org,
                             uint32_t seed, uint32_t* compared) {
    Scan S;
    const int rc = open_scan(file, len, S);
    if (rc) return -rc;
    auto word = [&](uint32_t b) {
        if ((b & 31u) || b - org > S.nbits + 4096u) __builtin_trap();
        return S.word((b - org) >> 5);
    };
    auto tab = [&](uint32_t k) { return S.y.sync_entry_at(k); };
    auto rows = [&](uint32_t k) { return S.y.sync_row_at(k); };
    auto bword = [&](uint32_t k) { return k < S.bmap.size() ? S.bmap[k] : 0u; };
    auto plain = plain_scan(S.y.units, S.y.upm, S.y.t.lut.data(), [&](uint32_t p) { return S.peek(p); });
    const bool restart = S.in.restart_interval != 0;
    Random rnd(seed);
    int bad = 0;
    *compared = 0;
    for (uint32_t k = 0; k < tries; ++k) {
        const uint32_t nsub = (S.nbits + L - 1) / L, i0 = rnd(nsub);
        PlainLane a;
        a.p = i0 * L + (rnd(4) ? rnd(31) : 0u);
        if (a.p >= S.nbits || (org >> 31 && a.p + org >= org)) continue;   // (a negative org: the stretch starts at bit -org)
        a.u = rnd(S.y.upm); a.z = rnd(3) ? rnd(64) : 0u;
        SyncLane b;
        sync_start(b, a.p + org, a.u, a.z, S.y.upm, kRow0, word, tab, rows);
        for (uint32_t i = i0; i < i0 + spans && i < nsub; ++i) {
            const uint32_t limit = (i + 1) * L;
            int64_t da = 0, db = 0;
            uint32_t ca = 0, cb = 0;
            a.nb = b.nb = 0;
            if (restart) {
                plain.sync_rst(a, limit, da, ca, bword);
                sync_span_rst(b, limit + org, db, cb, org, [&](uint32_t p) { sync_start(b, p, 0u, 0u, S.y.upm, kRow0, word, tab, rows); },
                              [&](uint32_t to) { sync_span(b, to, db, word, tab, rows); }, bword);
            } else {
                plain.sync(a, limit, da);
                sync_span(b, limit + org, db, word, tab, rows);
            }
            ++*compared;
            if (sync_pos(b) - org != a.p || S.y.unit_of_row(b.row) != a.u || ((b.S >> 9) & 63u) != a.z || a.nb != b.nb || da != db || ca != cb) { ++bad; break; }
        }
    }
    return bad;
}

// The write pass's lanes from `tries` states: what they store, unit, position, state, predictors and flags must be those of
// the plain ones.  States: random ones, and with `chain` those the true chain passes through (both flag nothing there).
// Predictors are compared in scans without intervals: a lane that has moved to the start of one has yet to clear them.
// total: units after which they stop (0: all of the image).
extern "C" int write_vs_plain(const uint8_t* file, size_t len, uint32_t L, uint32_t tries, int chain, uint32_t org, uint32_t total,
                              uint32_t seed, uint32_t* stored) {
    Scan S;
    const int rc = open_scan(file, len, S);
    if (rc) return -rc;
    auto word = [&](uint32_t b) {
        if ((b & 31u) || b - org > S.nbits + 4096u) __builtin_trap();
        return S.word((b - org) >> 5);
    };
    auto tab = [&](uint32_t k) { return S.y.write_entry_at(k); };
    auto rows = [&](uint32_t k) { return S.y.write_row_at(k); };
    auto bword = [&](uint32_t k) { return k < S.bmap.size() ? S.bmap[k] : 0u; };
    auto plain = plain_scan(S.y.units, S.y.upm, S.y.t.lut.data(), [&](uint32_t p) { return S.peek(p); });
    const uint32_t upm = S.y.upm;
    const bool restart = S.in.restart_interval != 0;
    const uint32_t upi = S.in.restart_interval * upm;
    Random rnd(seed);
    int bad = 0;
    *stored = 0;
    PlainLane c = {0u, 0u, 0u, 0u};   // the true chain
    const uint32_t nsub = (S.nbits + L - 1) / L;
    if (!total) total = S.in.total_units;
    for (uint32_t k = 0; k < tries && (!chain || k < nsub); ++k) {
        const uint32_t i = chain ? k : rnd(nsub), limit = (i + 1) * L;
        PlainLane a;
        a.p = chain ? c.p : i * L + rnd(31);
        a.u = chain ? c.u : rnd(upm);
        a.z = chain ? c.z : rnd(3) ? rnd(64) : 0u;
        a.nb = 0;
        const PlainLane in = a;
        // (no lane starts in the padding in front of an interval)
        const bool padding = restart && next_boundary(a.p, a.p + 8u, bword) != kNoBoundary && next_boundary(a.p, a.p + 8u, bword) > a.p;
        if (a.p < S.nbits && !(org >> 31 && a.p + org >= org) && !padding) {
            const uint32_t unit = chain ? c.nb : rnd(S.in.total_units) / upm * upm + a.u;
            const int32_t d[3] = {(int32_t)rnd(4096) - 2048, (int32_t)rnd(4096) - 2048, (int32_t)rnd(4096) - 2048};
            std::vector<std::pair<uint64_t, int>> sa, sb;
            uint32_t ua = unit, fa = 0, fb = 0;
            int32_t pred[3] = {d[0], d[1], d[2]};
            auto store_a = [&](uint32_t u, uint32_t at, int16_t v) { sa.push_back({(uint64_t)u * 64 + at, v}); };
            if (restart) plain.write_rst(a, limit, ua, total, upi, pred, store_a, fa, bword);
            else plain.write(a, limit, ua, total, pred, store_a, fa);
            WriteLane b;
            b.unit = unit;
            b.seen = 0;
            auto store_b = [&](uint32_t u, uint32_t at, int16_t v) { if (at > 63u) __builtin_trap(); sb.push_back({(uint64_t)u * 64 + at, v}); };
            write_predictors(b, S.y.component(in.u), d[0], d[1], d[2]);
            write_start(b, in.p + org, in.u, in.z, upm, kRow0, word, tab, rows);
            if (restart) write_span_rst(b, limit + org, total, upi, org, upm, kRow0, word, tab, rows, store_b, bword, &fb);
            else write_span(b, limit + org, total, word, tab, rows, store_b);
            if (b.seen & kWriteBad) fb |= kStInvalid;
            const uint32_t u = S.y.unit_of_row(b.s.row), z = (b.s.S >> 9) & 63u;
            WriteLane want = b;
            write_predictors(want, S.y.component(a.u), pred[0], pred[1], pred[2]);
            if (sa != sb || ua != b.unit || fa != fb || sync_pos(b.s) - org != a.p || u != a.u || z != a.z || (chain && fa) ||
                (!restart && (want.p0 != b.p0 || want.p1 != b.p1 || want.p2 != b.p2)))
                ++bad;
            // the values in chunks: nothing outside the image, whole chunks only from the lane's first slot on
            const uint32_t slots = total * 64u, first = unit * 64u + in.z;
            WriteChunk ch = chunk_start(first);
            std::map<uint64_t, int> put;
            auto store1 = [&](uint32_t at, int16_t v) { at < slots ? (void)(put[at] = v) : (void)++bad; };
            auto store8 = [&](uint32_t at, uint64_t a) {
                if ((at & 3u) || at > slots - 4u || (at < first && (!restart || chain))) ++bad;
                else for (uint32_t j = 0; j < 4u; ++j) put[at + j] = (int16_t)(uint16_t)(a >> (16u * j));
            };
            for (auto& v : sb) chunk_value(ch, (uint32_t)v.first, (int16_t)v.second, store8);
            chunk_ends(ch, store1);
            if (!restart || chain) {   // (from any state a lane may take a unit for the first of an interval, and store it twice)
                for (auto& v : sb) { bad += v.second != 0 && put[v.first] != v.second; put.erase(v.first); }
                for (auto& v : put) bad += v.second != 0;
            }
            *stored += (uint32_t)sb.size();
        }
        if (chain) {
            int64_t dc = 0;
            uint32_t crossed = 0;
            if (restart) plain.sync_rst(c, limit, dc, crossed, bword);
            else plain.sync(c, limit, dc);
        }
    }
    return bad;
}

// Position, unit and zig-zag index say all about a decoder: a lane that goes on and one that starts from them again, after
// every single symbol, read and store the same.  From `tries` random states, `symbols` symbols each; *compared: symbols.
extern "C" int lanes_restarted(const uint8_t* file, size_t len, uint32_t tries, uint32_t symbols, uint32_t seed, uint32_t* compared) {
    Scan S;
    const int rc = open_scan(file, len, S);
    if (rc) return -rc;
    auto word = [&](uint32_t b) { return S.word(b >> 5); };
    auto tab = [&](uint32_t k) { return S.y.sync_entry_at(k); };
    auto wtab = [&](uint32_t k) { return S.y.write_entry_at(k); };
    auto rows = [&](uint32_t k) { return S.y.sync_row_at(k); };
    auto wrows = [&](uint32_t k) { return S.y.write_row_at(k); };
    const uint32_t upm = S.y.upm;
    Random rnd(seed);
    auto unit_of = [&](const SyncLane& l) { return S.y.unit_of_row(l.row); };
    int bad = 0;
    *compared = 0;
    for (uint32_t k = 0; k < tries; ++k) {
        SyncLane a, b;
        WriteLane x, y;
        const uint32_t p0 = rnd(S.nbits), u0 = rnd(upm), z0 = rnd(2) ? rnd(64) : 0u;
        sync_start(a, p0, u0, z0, upm, kRow0, word, tab, rows);
        write_start(x, p0, u0, z0, upm, kRow0, word, wtab, wrows);
        for (uint32_t i = 0; i < symbols && sync_pos(a) < S.nbits; ++i, ++*compared) {
            const uint32_t p = sync_pos(a);
            int64_t da = 0, db = 0;
            a.nb = b.nb = 0;
            sync_start(b, p, unit_of(a), (a.S >> 9) & 63u, upm, kRow0, word, tab, rows);
            sync_span(a, p + 1u, da, word, tab, rows);
            sync_span(b, p + 1u, db, word, tab, rows);
            bad += a.S != b.S || sync_pos(a) != sync_pos(b) || a.row != b.row || a.nb != b.nb || da != db;
            std::vector<std::pair<uint32_t, int>> sx, sy;
            x.unit = y.unit = x.seen = y.seen = 0u;
            x.p0 = x.p1 = x.p2 = y.p0 = y.p1 = y.p2 = 0;
            write_start(y, p, unit_of(x.s), (x.s.S >> 9) & 63u, upm, kRow0, word, wtab, wrows);
            write_span(x, p + 1u, 2u, word, wtab, wrows, [&](uint32_t u, uint32_t at, int16_t v) { sx.push_back({u * 64u + at, v}); });
            write_span(y, p + 1u, 2u, word, wtab, wrows, [&](uint32_t u, uint32_t at, int16_t v) { sy.push_back({u * 64u + at, v}); });
            bad += sx != sy || x.seen != y.seen || x.s.S != a.S || y.s.S != a.S || x.s.row != a.row || sync_pos(x.s) != sync_pos(a);
        }
    }
    return bad;
}

// The walk of a whole wavefront from `tries` random states over `spans` subsequences of L bits against sync_span: mismatches in
// state, unit count and DC sums (where those fit the fields they are kept in).  *kinds: of data units.
extern "C" int walk_vs_lanes(const uint8_t* file, size_t len, uint32_t L, uint32_t tries, uint32_t spans, uint32_t seed,
                             uint32_t* compared, uint32_t* kinds) {
    Scan S;
    const int rc = open_scan(file, len, S);
    if (rc) return -rc;
    auto word = [&](uint32_t b) { return S.word(b >> 5); };
    auto tab = [&](uint32_t k) { return S.y.sync_entry_at(k); };
    auto rows = [&](uint32_t k) { return S.y.sync_row_at(k); };
    const uint32_t upm = S.y.upm;
    const Walk w = make_walk(S.y.walk, S.y.sched_comp, upm, S.y.t.ndc, kBase);
    *kinds = 0;
    for (uint32_t u = 0; u < upm; ++u) *kinds = std::max(*kinds, ((S.y.walk >> (2u * u)) & 3u) + 1u);
    Random rnd(seed);
    int bad = 0;
    *compared = 0;
    for (uint32_t k = 0; k < tries; ++k) {
        const uint32_t nsub = (S.nbits + L - 1) / L, i0 = rnd(nsub);
        uint32_t p = i0 * L + (rnd(4) ? rnd(31) : 0u), u = rnd(upm), z = rnd(3) ? rnd(64) : 0u;
        SyncLane b;
        sync_start(b, p, u, z, upm, kRow0, word, tab, rows);
        for (uint32_t i = i0; i < i0 + spans && i < nsub; ++i, ++*compared) {
            uint32_t nb;
            int64_t da, db = 0;
            int32_t exact[3];
            b.nb = 0;
            walk_span(p, u, z, nb, da, exact, (i + 1) * L, w, word, tab);
            sync_span(b, (i + 1) * L, db, word, tab, rows);
            const bool fits = std::abs(exact[0]) < 16384 && std::abs(exact[1]) < 16384 && std::abs(exact[2]) < 16384;
            if (p != sync_pos(b) || u != S.y.unit_of_row(b.row) || z != ((b.S >> 9) & 63u) || nb != b.nb || (fits && da != db)) { ++bad; break; }
        }
    }
    return bad;
}

// Every 16-bit stretch looked up in a table of build_lut and in its layout for the synchronisation kernels: mismatches.
extern "C" int sync_table_vs_lut(const uint8_t* bits, const uint8_t* vals, int is_dc) {
    Tables t;
    t.ndc = is_dc ? 1u : 0u;
    t.nslots = 1u;
    t.lut.assign(kLutEntries, 0);
    if (!build_lut(bits, vals, is_dc != 0, t.lut.data())) return -1;
    if (!lay_out<false>(t, kBase, t.sync) || !lay_out<true>(t, kBase, t.write)) return -2;
    int bad = 0;
    for (uint32_t v = 0; v < 65536u; ++v) {
        const uint32_t peek = v << 16 | 0x5A5Au;
        uint32_t e = t.lut[peek >> (32 - kLutK)];
        if (lut_esc(e)) {
            const uint32_t n = lut_esc_bits(e);
            e = t.lut[kLutL1 + lut_esc_offset(e) + ((peek >> (32 - kLutK - n)) & ((1u << n) - 1u))];
        }
        uint32_t s = t.sync.at(peek >> (32u - (is_dc ? kSyncDcK : kSyncAcK)));
        if (s & kSyncEsc) {
            const uint32_t k = sync_escape_at(s, peek);
            if (k < kBase || (k & 3u)) return -3;
            s = t.sync.at((k - kBase) / 4);
        }
        uint32_t w = t.write.at(peek >> (32u - (is_dc ? kSyncDcK : kSyncAcK)));
        if (w & kSyncEsc) w = t.write.at((sync_escape_at(w, peek) - kBase) / 4);
        const bool inside = !is_dc && lut_adv(e) != 0u && lut_adv(e) != kAdvEob;
        const uint32_t slots = lut_adv(e);
        const bool coded = is_dc ? slots == 1u : slots != 0u;
        bad += (is_dc && slots != 1u && slots != 2u) || w != ((e & 31u) | slots << 9 | lut_size(e) << 20 | (inside ? kWriteInside : 0u) | (coded ? 0u : kWriteNoCode) |
                    (!coded ? 0u : is_dc ? 3u << 29 : lut_size(e) ? 1u << 30 : 0u));
        bad += (s & 31u) != lut_total(e) || ((s >> 9) & 63u) != slots || ((s >> 20) & 15u) != (is_dc ? lut_size(e) : 0u) || (s & 0x81E0u);
    }
    return bad;
}
