// Host walk-through of the decoder's kernels: the lanes on the kernels' tables (sync_span, write_span and their _rst forms of
// jpgd_lane.h, which the kernels have in assembly), the walk of a whole wavefront (jpgd_walk.h) and the same index arithmetic
// as jpgd_kernels.h, with workgroups and lanes run one after another.
// It exists so that the CPU-only test run can check the host logic (tables, lane decoder, record
// packing, padded staging layout, scan, write, pixel arithmetic) before anything reaches a GPU.
// It is test code: the library never calls it and it is not a fallback for the GPU path.
//
// Build: g++ -O2 -std=c++17 -shared -fPIC -o libjpgd_emul.so jpgd_emul.cpp ../../paper_2111_09219_amd/csrc/jpgd_parse.cpp
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../paper_2111_09219_amd/csrc/jpgd_idct.h"
#include "jpgd_tables.h"
#include "jpgd_walk.h"

using namespace jpgd;

namespace {

uint32_t bswap(uint32_t v) { return __builtin_bswap32(v); }
int32_t sx16(uint32_t v) { return (int32_t)(int16_t)(v & 0xFFFFu); }
uint32_t pack_dc01(int64_t acc) { int32_t a, b, c; dc_unpack(acc, a, b, c); return ((uint32_t)a & 0xFFFFu) | ((uint32_t)b << 16); }
uint32_t pack_dc2(int64_t acc) { int32_t a, b, c; dc_unpack(acc, a, b, c); return (uint32_t)c & 0xFFFFu; }

struct Image {
    jpgd_info in;
    Layout y;
    std::vector<uint8_t> stream;  // unstuffed + zero slack
    std::vector<uint32_t> bmap;   // restart intervals: one bit per unstuffed byte, set at the first byte of an interval
    uint32_t nbytes = 0, nsub = 0, markers = 0;
};

int prepare(const uint8_t* file, size_t len, Image& im) {
    const int rc = jpgd_parse(file, len, &im.in);
    return rc ? rc : make_layout(im.in, im.y);
}

// the two unstuff kernels, tile by tile and lane by lane
void unstuff(const uint8_t* scan, uint32_t n, uint32_t logL, Image& im) {
    const uint32_t tiles = (n + kUnstuffTile - 1) / kUnstuffTile;
    const bool restart = im.in.restart_interval != 0;
    std::vector<uint32_t> removed(tiles, 0), before(tiles, 0);
    auto keep_mask = [&](uint32_t pos, uint32_t& nvalid, uint32_t& marks) {
        nvalid = pos >= n ? 0u : std::min(16u, n - pos);
        uint32_t prev = (pos > 0 && nvalid) ? scan[pos - 1] : 0u, mask = 0;
        marks = 0;
        for (uint32_t j = 0; j < nvalid; ++j) {
            uint32_t b = scan[pos + j];
            bool nx_exists = pos + j + 1 < n;
            uint32_t nx = nx_exists ? scan[pos + j + 1] : 0u;
            bool rst2 = restart && prev == 255 && (b & 0xF8) == 0xD0;
            bool rst1 = restart && b == 255 && nx_exists && (nx & 0xF8) == 0xD0;
            if (!((b == 0 && prev == 255) || rst1 || rst2)) mask |= 1u << j;
            if (rst2) marks |= 1u << j;
            prev = b;
        }
        return mask;
    };
    im.markers = 0;
    for (uint32_t t = 0; t < tiles; ++t)
        for (uint32_t lane = 0; lane < (uint32_t)kWG; ++lane) {
            uint32_t nv, mk, m = keep_mask(t * kUnstuffTile + lane * 16, nv, mk);
            removed[t] += nv - (uint32_t)__builtin_popcount(m);
            im.markers += (uint32_t)__builtin_popcount(mk);
        }
    uint32_t carry = 0;
    for (uint32_t t = 0; t < tiles; ++t) { before[t] = carry; carry += removed[t]; }
    im.nbytes = n - carry;
    const uint32_t L = 1u << logL;
    im.nsub = (uint32_t)(((uint64_t)im.nbytes * 8 + L - 1) >> logL);
    im.stream.assign((size_t)n + L / 8 + 64 + 16 + 256, 0xAA);  // poison: the kernels must define what they read
    im.bmap.assign((size_t)tiles * 128 + 128, 0);
    for (uint32_t t = 0; t < tiles; ++t) {
        uint32_t o = t * kUnstuffTile - before[t];
        for (uint32_t lane = 0; lane < (uint32_t)kWG; ++lane) {
            uint32_t pos = t * kUnstuffTile + lane * 16, nv, mk, m = keep_mask(pos, nv, mk);
            for (uint32_t j = 0; j < nv; ++j) {
                if (mk & (1u << j)) im.bmap[o >> 5] |= 1u << (o & 31);  // the next kept byte starts an interval
                if (m & (1u << j)) im.stream[o++] = scan[pos + j];
            }
        }
    }
    for (uint32_t k = 0; k < L / 8 + 64; ++k) im.stream[im.nbytes + k] = 0;
}

struct Emul {
    Image im;
    uint32_t logL, H, seq_len;
    std::vector<SInfo> sinfo;
    std::vector<uint32_t> warm;  // per sequence: the state its records continue (0xFFFFFFFF = none)
    Walk walk;
    uint32_t inter_changed = 0, rounds_max = 0, flags = 0, pending = 0;
};

uint32_t g_coop_max = kCoopMax;  // as the library sets it for four wavefronts; the tests also run with 0 (never), 8 and 64
uint32_t g_sync_waves = kWG / 64;  // wavefronts per workgroup (the library launches 4, 8 or 16)

constexpr uint32_t kStreamAt = 4096;  // byte of LDS at which the stream lies
constexpr uint32_t kPadWords = 12;     // behind it, for what the walk looks at

void sync_intra(Emul& E) {
    const Image& im = E.im;
    const uint32_t nsub = im.nsub, logL = E.logL, L = 1u << logL, wps = L >> 5;
    const uint32_t nseq = (nsub + E.seq_len - 1) / E.seq_len;
    const uint32_t* words = (const uint32_t*)im.stream.data();
    std::vector<uint32_t> strm;
    for (uint32_t wg = 0; wg < nseq; ++wg) {
        const int32_t base = (int32_t)(wg * E.seq_len) - (int32_t)E.H;
        const uint32_t first = base < 0 ? 0u : (uint32_t)base;
        const uint32_t t0 = (uint32_t)((int32_t)first - base);
        const uint32_t t1 = std::min<uint32_t>(kWG, (uint32_t)((int32_t)nsub - base));
        const uint32_t first_word = first * wps, nwords = (t1 - t0) * wps + 4;
        strm.assign(nwords + kPadWords, 0xDEADBEEF);
        for (uint32_t r = 0; r < nwords; ++r) strm[r] = bswap(words[first_word + r]);
        // the lanes' bits count from where the stream lies in LDS
        const uint32_t org = 8 * kStreamAt - (first_word << 5);
        auto staged = [&](uint32_t b, uint32_t n) {
            if ((b & 31) || b / 32 - kStreamAt / 4 >= n) abort();  // a lane looked outside the staged stretch
            return strm[b / 32 - kStreamAt / 4];
        };
        auto word = [&](uint32_t b) { return staged(b, nwords); };
        auto walk_word_at = [&](uint32_t p) { return staged(p + org, nwords + kPadWords); };
        auto tab = [&](uint32_t k) { return im.y.sync_entry_at(k); };
        auto rows = [&](uint32_t k) { return im.y.sync_row_at(k); };
        // the part of the bitmap the kernel stages with these words
        const bool restart = im.in.restart_interval != 0;
        const uint32_t bm_k0 = first_word >> 3, bm_n = ((first_word + nwords + 7) >> 3) - bm_k0 + 1;
        auto bword = [&](uint32_t k) {
            if (k < bm_k0 || k - bm_k0 >= bm_n) abort();  // a lane looked outside the staged bitmap
            return im.bmap[k];
        };
        uint32_t sw[kWG], pnb[kWG], pdc01[kWG], pdc2[kWG];
        SyncLane l[kWG];
        bool active[kWG];
        uint32_t tt[kWG], chain[kWG] = {0};  // chain: state in front of its target, once chains have a wavefront each
        auto start_of = [&](uint32_t k) { return (uint32_t)(base + (int32_t)k) << logL; };
        auto state_of = [&](const SyncLane& a, uint32_t end) { return pack_state(sync_pos(a) - org - end, (a.S >> 9) & 63u, im.y.unit_of_row(a.row)); };
        auto start = [&](SyncLane& a, uint32_t p, uint32_t u, uint32_t z) { sync_start(a, p + org, u, z, im.y.upm, kRow0, word, tab, rows); };
        auto decode = [&](SyncLane& a, uint32_t limit, int64_t& dc, uint32_t& crossed) {
            a.nb = 0;
            if (restart)
                sync_span_rst(a, limit + org, dc, crossed, org, [&](uint32_t p) { sync_start(a, p, 0u, 0u, im.y.upm, kRow0, word, tab, rows); },
                              [&](uint32_t to) { sync_span(a, to, dc, word, tab, rows); }, bword);
            else sync_span(a, limit + org, dc, word, tab, rows);
        };
        auto put_record = [&](uint32_t k, uint32_t x, uint32_t nb, uint32_t crossed, int64_t dc) {
            if (nb > 0x7FFFu) abort();  // records in LDS have 15 bits for the units
            sw[k] = x; pnb[k] = nb | (crossed << 31); pdc01[k] = pack_dc01(dc); pdc2[k] = pack_dc2(dc);
        };
        for (uint32_t t = 0; t < (uint32_t)kWG; ++t) {
            active[t] = false;
            if (t < t0 || t >= t1) continue;
            int64_t dc = 0;
            uint32_t crossed = 0;
            start(l[t], start_of(t), 0, 0);
            decode(l[t], start_of(t + 1), dc, crossed);
            put_record(t, state_of(l[t], start_of(t + 1)), l[t].nb, crossed, dc);
            active[t] = t + 1 < t1;
            tt[t] = t + 1;
        }
        uint32_t rounds = 0, waves_used = kWG / 64;
        bool coop = false;
        for (;;) {
            uint32_t now = 0;
            for (uint32_t t = 0; t < (uint32_t)kWG; ++t) now += active[t] ? 1u : 0u;
            if (!now) break;
            ++rounds;
            if (!coop && now <= (restart ? std::min(g_coop_max, g_sync_waves) : g_coop_max)) {
                coop = true;  // from here on a wavefront per chain
                for (uint32_t t = 0; t < (uint32_t)kWG; ++t)
                    if (active[t]) chain[t] = state_of(l[t], start_of(tt[t]));
            }
            // the chains move together where that frees a wavefront; in between a lane goes on with its own
            const bool packed = !coop && ((now + 63u) >> 6) < waves_used;
            if (packed) waves_used = (now + 63u) >> 6;
            for (uint32_t t = 0; t < (uint32_t)kWG; ++t) {
                if (!active[t]) continue;
                const uint32_t limit = start_of(tt[t] + 1);
                int64_t dc = 0;
                uint32_t x, nb, crossed = 0;
                if (packed) {
                    const uint32_t m = state_of(l[t], start_of(tt[t]));
                    start(l[t], start_of(tt[t]) + state_prel(m), state_u(m), state_z(m));
                }
                uint32_t p = start_of(tt[t]) + state_prel(chain[t]), u = state_u(chain[t]), z = state_z(chain[t]);
                // (a chain whose stretch holds an interval start is decoded by one lane with the interval rules)
                if (coop && (!restart || next_boundary(p, limit + 64u, bword) == kNoBoundary)) {
                    int32_t exact[3];
                    walk_span(p, u, z, nb, dc, exact, limit, E.walk, walk_word_at, tab);
                    x = pack_state(p - limit, z, u);
                } else {
                    if (coop) start(l[t], p, u, z);
                    decode(l[t], limit, dc, crossed);
                    x = state_of(l[t], limit);
                    nb = l[t].nb;
                }
                const bool synced = x == sw[tt[t]];
                put_record(tt[t], x, nb, crossed, dc);
                chain[t] = x;
                ++tt[t];
                active[t] = !synced && tt[t] < t1;
            }
        }
        E.rounds_max = std::max(E.rounds_max, rounds);
        E.warm[wg] = (E.H > 0 && E.H - 1 >= t0) ? sw[E.H - 1] : 0xFFFFFFFFu;
        for (uint32_t t = std::max(t0, E.H); t < t1; ++t) {
            SInfo r = {sw[t], pnb[t], pdc01[t], pdc2[t]};
            E.sinfo[(uint32_t)(base + (int32_t)t)] = r;
        }
    }
}

void sync_inter(Emul& E) {
    const Image& im = E.im;
    const uint32_t nsub = im.nsub, logL = E.logL;
    const uint32_t* words = (const uint32_t*)im.stream.data();
    auto word = [&](uint32_t b) { return b / 32 < im.stream.size() / 4 ? bswap(words[b / 32]) : 0u; };
    auto tab = [&](uint32_t k) { return im.y.sync_entry_at(k); };
    auto rows = [&](uint32_t k) { return im.y.sync_row_at(k); };
    auto bword = [&](uint32_t k) { return im.bmap[k]; };
    const bool restart = im.in.restart_interval != 0;
    E.inter_changed = 0;
    // On the GPU all boundaries are looked at together: every lane reads the last record of the sequence before
    // its boundary when the kernel starts, whatever another lane does to that record later in the same round.
    std::vector<uint32_t> seen;
    for (uint32_t b = 0; (uint64_t)(b + 1) * E.seq_len < nsub; ++b) seen.push_back(E.sinfo[(b + 1) * E.seq_len - 1].x);
    const std::vector<uint32_t> at_start = E.warm;
    for (uint32_t b = 0;; ++b) {
        uint64_t gfirst = (uint64_t)(b + 1) * E.seq_len;
        if (gfirst >= nsub) break;
        uint32_t g = (uint32_t)gfirst, gend = std::min(nsub, g + E.seq_len);
        uint32_t x0 = seen[b];
        if (E.warm[b + 1] == x0) continue;  // the two sequences already form one chain
        // few of the 64 boundaries of a workgroup to decode from: the wavefront walks them one after the other
        uint32_t workers = 0;
        for (uint32_t k = b & ~63u; k < std::min<uint32_t>((b & ~63u) + 64u, (uint32_t)seen.size()); ++k) workers += at_start[k + 1] != seen[k];
        const bool walks = !restart && workers <= (uint32_t)kInterCoopMax;
        uint32_t p = (g << logL) + state_prel(x0), u = state_u(x0), z = state_z(x0);
        SyncLane l;
        sync_start(l, p, u, z, im.y.upm, kRow0, word, tab, rows);
        bool first = true;
        for (;;) {
            int64_t dc = 0;
            const uint32_t limit = (g + 1) << logL;
            uint32_t crossed = 0, nb, x;
            if (walks) {
                int32_t exact[3];
                walk_span(p, u, z, nb, dc, exact, limit, E.walk, word, tab);
                x = pack_state(p - limit, z, u);
            } else {
                l.nb = 0;
                if (restart)
                    sync_span_rst(l, limit, dc, crossed, 0u, [&](uint32_t q) { sync_start(l, q, 0u, 0u, im.y.upm, kRow0, word, tab, rows); },
                                  [&](uint32_t to) { sync_span(l, to, dc, word, tab, rows); }, bword);
                else sync_span(l, limit, dc, word, tab, rows);
                nb = l.nb;
                x = pack_state(sync_pos(l) - limit, (l.S >> 9) & 63u, im.y.unit_of_row(l.row));
            }
            const bool synced = x == E.sinfo[g].x;
            if (first && !synced) E.inter_changed++;
            first = false;
            E.sinfo[g] = SInfo{x, nb | (crossed << 31), pack_dc01(dc), pack_dc2(dc)};
            ++g;
            if (synced || g >= gend) break;
        }
        E.warm[b + 1] = x0;
    }
}

// k_group_totals: does every sequence's set of records continue the state the sequence before it ends in?
void check_boundaries(Emul& E) {
    E.pending = 0;
    for (uint32_t b = 0; (uint64_t)(b + 1) * E.seq_len < E.im.nsub; ++b)
        if (E.warm[b + 1] != E.sinfo[(b + 1) * E.seq_len - 1].x) E.pending = 1;
}

void scan_and_write(Emul& E, int16_t* coef) {
    const Image& im = E.im;
    const uint32_t nsub = im.nsub, logL = E.logL, L = 1u << logL, wps = L >> 5;
    const uint32_t total = im.in.total_units;
    // poison: every coefficient has to be cleared by the group whose range holds it
    for (size_t k = 0; k < (size_t)total * 64; ++k) coef[k] = 0x5A5A;
    std::vector<uint8_t> cleared((size_t)total * 64, 0);
    const uint32_t* words = (const uint32_t*)im.stream.data();
    uint32_t unit0 = 0;
    int32_t pred[3] = {0, 0, 0};
    std::vector<uint32_t> strm;
    E.flags = 0;
    for (uint32_t i0 = 0; i0 < nsub; i0 += kWG) {
        const uint32_t nloc = std::min<uint32_t>(kWG, nsub - i0);
        const uint32_t first_word = i0 * wps, nwords = nloc * wps + 4;
        strm.assign(nwords, 0xDEADBEEF);
        for (uint32_t r = 0; r < nwords; ++r) strm[r] = bswap(words[first_word + r]);
        const uint32_t org = 8 * kStreamAt - (first_word << 5);
        auto word = [&](uint32_t b) {
            if ((b & 31) || b / 32 - kStreamAt / 4 >= nwords) abort();
            return strm[b / 32 - kStreamAt / 4];
        };
        auto tab = [&](uint32_t k) { return im.y.write_entry_at(k); };
        auto rows = [&](uint32_t k) { return im.y.write_row_at(k); };
        const bool restart = im.in.restart_interval != 0;
        const uint32_t bm_k0 = first_word >> 3, bm_n = ((first_word + nwords + 7) >> 3) - bm_k0 + 1;
        auto bword = [&](uint32_t k) {
            if (k < bm_k0 || k - bm_k0 >= bm_n) abort();
            return im.bmap[k];
        };
        {
            uint32_t grp_units = 0;
            for (uint32_t t = 0; t < nloc; ++t) grp_units += rec_units(E.sinfo[i0 + t].y);
            const uint64_t end_all = (uint64_t)total * 64;
            const uint32_t x_in = i0 ? E.sinfo[i0 - 1].x : 0u, x_out = E.sinfo[i0 + nloc - 1].x;
            uint64_t a = (uint64_t)unit0 * 64 + state_z(x_in);
            uint64_t b = i0 + nloc >= nsub ? end_all : ((uint64_t)unit0 + grp_units) * 64 + state_z(x_out);
            if (i0 == 0) a = 0;
            if (b > end_all) b = end_all;
            for (uint64_t k = a; k < b; ++k) {
                if (cleared[k]) abort();  // ranges of different groups must not overlap
                cleared[k] = 1;
                coef[k] = 0;
            }
        }
        const uint32_t grp_slot = unit0 * 64u;
        for (uint32_t t = 0; t < nloc; ++t) {
            const uint32_t i = i0 + t;
            const SInfo mine = E.sinfo[i];
            const uint32_t xprev = i ? E.sinfo[i - 1].x : 0u;
            const uint32_t u_in = state_u(xprev), z_in = state_z(xprev);
            uint32_t flags = 0;
            if (unit0 < total && unit0 % im.in.units_per_mcu != u_in) flags |= kStUnit;
            const uint32_t limit = (i + 1) << logL;
            WriteLane l;
            l.unit = unit0;
            l.seen = 0;
            write_predictors(l, im.y.component(u_in), (int16_t)pred[0], (int16_t)pred[1], (int16_t)pred[2]);
            // the values leave in chunks of four slots, counted from the first unit of the group
            WriteChunk chunk = chunk_start(unit0 * 64u + z_in - grp_slot);
            auto put = [&](uint32_t slot, int16_t v) {
                if ((uint64_t)grp_slot + slot >= (uint64_t)total * 64) abort();
                coef[(size_t)grp_slot + slot] = v;
            };
            auto store8 = [&](uint32_t slot, uint64_t v) { for (uint32_t k = 0; k < 4; ++k) put(slot + k, (int16_t)(uint16_t)(v >> (16 * k))); };
            auto store = [&](uint32_t k, uint32_t at, int16_t v) {
                if (k >= total || at > 63) abort();
                chunk_value(chunk, k * 64u + at - grp_slot, v, store8);
            };
            if (unit0 < total) {
                write_start(l, (i << logL) + state_prel(xprev) + org, u_in, z_in, im.y.upm, kRow0, word, tab, rows);
                if (restart) write_span_rst(l, limit + org, total, im.in.restart_interval * im.in.units_per_mcu, org, im.y.upm, kRow0, word, tab, rows, store, bword, &flags);
                else write_span(l, limit + org, total, word, tab, rows, store);
            }
            if (l.seen & kWriteBad) flags |= kStInvalid;
            chunk_ends(chunk, put);
            if (restart && i == 0) {
                const uint64_t mcus = (uint64_t)im.in.mcus_x * im.in.mcus_y;
                if (im.markers != (uint32_t)((mcus + im.in.restart_interval - 1) / im.in.restart_interval) - 1) flags |= kStInvalid;
            }
            if (l.unit < total) {
                const uint32_t p = sync_pos(l.s) - org;
                if (p < limit || pack_state(p - limit, (l.s.S >> 9) & 63u, im.y.unit_of_row(l.s.row)) != mine.x) flags |= kStMismatch;
                if (i == nsub - 1) flags |= kStShort;
            }
            E.flags |= flags;
            // exclusive scan, lane by lane; the DC sums start afresh after a subsequence in which an interval began
            unit0 += rec_units(mine.y);
            if (rec_restarted(mine.y)) pred[0] = pred[1] = pred[2] = 0;
            pred[0] += sx16(mine.z); pred[1] += sx16(mine.z >> 16); pred[2] += sx16(mine.w);
        }
    }
}

void pixels(const Emul& E, const int16_t* coef_all, uint8_t* pix) {
    const jpgd_info& in = E.im.in;
    const uint8_t zz[64] = JPGD_ZIGZAG_LITERAL;
    const uint32_t upm = in.units_per_mcu, hs = in.hsamp[0], vs = in.vsamp[0], ncomp = in.ncomp;
    const uint32_t M = kPixBlocks / upm, runs = (in.mcus_x + M - 1) / M;
    const uint32_t mcu_w = 8 * hs, mcu_h = 8 * vs;
    std::vector<float> blk(kPixBlocks * 72);
    for (uint32_t mrow = 0; mrow < in.mcus_y; ++mrow)
        for (uint32_t run = 0; run < runs; ++run) {
            const uint32_t m0 = run * M, nm = std::min(M, in.mcus_x - m0), nblk = nm * upm;
            const int16_t* coef = coef_all + ((size_t)mrow * in.mcus_x + m0) * upm * 64;
            for (uint32_t k = 0; k < nblk; ++k) {
                uint32_t comp = E.im.y.component(k % upm);
                for (uint32_t zi = 0; zi < 64; ++zi)
                    blk[k * 72 + (zz[zi] >> 3) * 9 + (zz[zi] & 7)] = (float)coef[k * 64 + zi] * (float)in.qt[in.tq[comp]][zi];
            }
            for (uint32_t j = 0; j < nblk * 8; ++j) {
                float* b = &blk[(j >> 3) * 72 + (j & 7)];
                idct8(b[0], b[9], b[18], b[27], b[36], b[45], b[54], b[63]);
            }
            for (uint32_t j = 0; j < nblk * 8; ++j) {
                float* b = &blk[(j >> 3) * 72 + (j & 7) * 9];
                b[0] += kLevelShiftDc;
                idct8(b[0], b[1], b[2], b[3], b[4], b[5], b[6], b[7]);
            }
            for (uint32_t py = 0; py < mcu_h; ++py)
                for (uint32_t px = 0; px < nm * mcu_w; ++px) {
                    uint32_t gy = mrow * mcu_h + py, gx = m0 * mcu_w + px;
                    if (gy >= in.height || gx >= in.width) continue;
                    uint32_t m = px / mcu_w, xin = px % mcu_w;
                    float y = blk[(m * upm + (py >> 3) * hs + (xin >> 3)) * 72 + (py & 7) * 9 + (xin & 7)];
                    uint8_t* dst = pix + ((size_t)gy * in.width + gx) * ncomp;
                    if (ncomp == 1) { dst[0] = (uint8_t)pack_u8(y, 0u, 0u); continue; }
                    const float* cbb = &blk[(m * upm + hs * vs) * 72 + (py / vs) * 9];
                    const ChromaTerms c = chroma_terms(cbb[xin / hs], cbb[72 + xin / hs]);
                    dst[0] = (uint8_t)pack_u8(y + c.r, 0u, 0u);
                    dst[1] = (uint8_t)pack_u8(y + c.g, 0u, 0u);
                    dst[2] = (uint8_t)pack_u8(y + c.b, 0u, 0u);
                }
        }
}

}  // namespace

// Runs the whole pipeline on the host.  stats: [0] inter-sequence rounds used, [1] boundaries whose first
// comparison failed in the last round, [2] longest intra-sequence overflow (rounds), [3] final flags,
// [4] number of subsequences, [5] unstuffed bytes.  sinfo_out (may be NULL): 4 words per subsequence.
extern "C" int emul_decode(const uint8_t* file, size_t len, uint32_t L, uint32_t H, uint32_t max_rounds, int16_t* coef,
                           uint8_t* pix, uint32_t* sinfo_out, uint32_t sinfo_cap, uint8_t* stream_out,
                           uint32_t* stats) {
    Emul E;
    int rc = prepare(file, len, E.im);
    if (rc) return rc;
    E.logL = 0;
    while ((1u << E.logL) < L) ++E.logL;
    E.H = H;
    E.seq_len = kWG - H;
    E.walk = make_walk(E.im.y.walk, E.im.y.sched_comp, E.im.y.upm, E.im.y.t.ndc, kBase);
    unstuff(file + E.im.in.scan_offset, (uint32_t)E.im.in.scan_bytes, E.logL, E.im);
    E.sinfo.assign(E.im.nsub, SInfo{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu});
    const uint32_t nseq = (E.im.nsub + E.seq_len - 1) / E.seq_len;
    E.warm.assign(nseq + 1, 0xFFFFFFFFu);
    sync_intra(E);
    // as the host code of the library: everything once; if a boundary is still open, rounds that settle the
    // boundaries, then the write pass once more
    uint32_t rounds = 0;
    auto scan = [&]() {
        if (nseq > 1) { sync_inter(E); ++rounds; }
        check_boundaries(E);
    };
    scan();
    scan_and_write(E, coef);
    if (E.pending && nseq > 1 && rounds < max_rounds) {
        while (E.pending && rounds < max_rounds) scan();
        const bool open = E.pending != 0;
        scan_and_write(E, coef);
        if (open) E.flags |= kStMismatch;
    } else if (E.pending && nseq > 1) {
        E.flags |= kStMismatch;
    }
    if (stats) {
        stats[0] = rounds; stats[1] = E.inter_changed; stats[2] = E.rounds_max; stats[3] = E.flags;
        stats[4] = E.im.nsub; stats[5] = E.im.nbytes;
    }
    if (sinfo_out && sinfo_cap >= E.im.nsub) memcpy(sinfo_out, E.sinfo.data(), (size_t)E.im.nsub * 16);
    if (stream_out) memcpy(stream_out, E.im.stream.data(), E.im.nbytes);
    if (E.flags) return JPGD_E_CORRUPT;
    if (pix) pixels(E, coef, pix);
    return JPGD_OK;
}

// chains left at which the intra-sequence walk-through switches to the wavefront-per-chain decoder
extern "C" void emul_set_coop_max(uint32_t n) { g_coop_max = n; }
extern "C" void emul_set_sync_waves(uint32_t n) { g_sync_waves = n; }

// the literal zig-zag table of jpgd_idct.h, for comparison with a generated one
extern "C" void emul_zigzag(uint8_t out[64]) {
    const uint8_t zz[64] = JPGD_ZIGZAG_LITERAL;
    memcpy(out, zz, 64);
}

// the pixel kernel's choice between ordinary and streaming accesses
extern "C" int emul_pass_caches(uint64_t coef_and_pixel_bytes) { return pass_caches(coef_and_pixel_bytes) ? 1 : 0; }

// the write kernel's room for its output in LDS
extern "C" uint32_t emul_tile_room(uint32_t total_units, uint64_t scan_bytes, uint32_t L) { return tile_room(total_units, scan_bytes, L); }

// one table built by jpgd_lut.h
extern "C" int emul_build_lut(const uint8_t* bits, const uint8_t* vals, int is_dc, uint16_t* out) {
    return build_lut(bits, vals, is_dc != 0, out) ? 0 : JPGD_E_TABLE;
}

// pair bytes of an AC table built by jpgd_lut.h (lut: the table's kLutEntries entries)
extern "C" void emul_build_pairs(const uint16_t* lut, uint8_t* pairs) { build_pairs(lut, pairs); }

// The synchronisation pass with two symbols per step (sync_span) against the one with single symbols, from decoder states that
// need not lie on the true chain: `nstart` starts at pseudo-random subsequences in pseudo-random states, each
// followed over `span` subsequences by both decoders (the lanes keep their window from one subsequence to the
// next, as in the kernel's overflow rounds).  Returns the number of subsequences after which the two disagreed in
// position, unit, zig-zag index, completed units or DC sums; stats[0] = steps of the single decoder,
// stats[1] = steps of the pair decoder over the same stretches.
extern "C" int emul_pairs_vs_single(const uint8_t* file, size_t len, uint32_t L, uint32_t nstart, uint32_t span,
                                    uint32_t seed, uint32_t* stats) {
    Image im;
    if (prepare(file, len, im) || im.in.restart_interval) return -1;
    uint32_t logL = 0;
    while ((1u << logL) < L) ++logL;
    unstuff(file + im.in.scan_offset, (uint32_t)im.in.scan_bytes, logL, im);
    const uint32_t* words = (const uint32_t*)im.stream.data();
    uint32_t steps = 0;
    auto at = [&](uint32_t k) { return k < im.stream.size() / 4 ? bswap(words[k]) : 0u; };
    auto word = [&](uint32_t b) { ++steps; return at(b / 32); };  // one word per step (and up to three where a lane starts)
    auto tab = [&](uint32_t k) { return im.y.sync_entry_at(k); };
    auto rows = [&](uint32_t k) { return im.y.sync_row_at(k); };
    auto single = plain_scan(im.y.units, im.y.upm, im.y.t.lut.data(),
                             [&](uint32_t p) { return (uint32_t)((((uint64_t)at(p / 32) << 32 | at(p / 32 + 1)) << (p & 31u)) >> 32); });
    uint64_t rng = 0x9E3779B97F4A7C15ull ^ seed;
    auto next = [&]() { rng ^= rng << 13; rng ^= rng >> 7; rng ^= rng << 17; return (uint32_t)(rng >> 16); };
    int bad = 0;
    if (im.nsub < 2) return 0;
    for (uint32_t k = 0; k < nstart; ++k) {
        const uint32_t i0 = next() % (im.nsub - 1u);
        const uint32_t prel = next() % 32u, z = next() % 64u, u = next() % im.in.units_per_mcu;
        PlainLane a = {(i0 << logL) + prel, u, z, 0u};
        SyncLane b;
        sync_start(b, a.p, u, z, im.y.upm, kRow0, word, tab, rows);
        for (uint32_t i = i0; i < std::min(im.nsub, i0 + span); ++i) {
            const uint32_t limit = (i + 1u) << logL;
            int64_t da = 0, db = 0;
            a.nb = b.nb = 0;
            single.sync(a, limit, da);
            sync_span(b, limit, db, word, tab, rows);
            if (a.p != sync_pos(b) || a.u != im.y.unit_of_row(b.row) || a.z != ((b.S >> 9) & 63u) || a.nb != b.nb || da != db) { ++bad; break; }
        }
    }
    stats[0] = single.symbols;
    stats[1] = steps;
    return bad;
}
