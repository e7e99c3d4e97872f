// The lanes of the two passes in their plainest form: one symbol after the other, from the tables of jpgd_lut.h, bit positions
// and nothing kept from step to step but the state.  What the kernels' lanes (jpgd_lane.h) are held to.  Test code: the
// library never calls it.
#pragma once
#include "../../paper_2111_09219_amd/csrc/jpgd_lane.h"

namespace jpgd {

struct PlainUnit {
    uint32_t dc, ac;  // first entry of its tables in `lut`
    uint32_t comp;
};

struct PlainLane {
    uint32_t p;   // bit of the next symbol
    uint32_t u;   // data unit inside the MCU
    uint32_t z;   // zig-zag index of the next coefficient (0 = a DC symbol is next)
    uint32_t nb;  // data units completed since it was last cleared
};

// peek(p): the 32 bits from bit p on
template <class Peek>
struct PlainScan {
    const PlainUnit* units;
    uint32_t upm;
    const uint16_t* lut;
    Peek peek;
    uint32_t symbols = 0;  // taken so far

    struct Symbol {
        bool is_dc, coded, done;
        uint32_t u, z, size, slots;
        int32_t value;
    };
    Symbol next(PlainLane& l) {
        const PlainUnit& unit = units[l.u];
        Symbol s;
        s.is_dc = l.z == 0u;
        s.u = l.u;
        s.z = l.z;
        const uint32_t bits = peek(l.p), table = s.is_dc ? unit.dc : unit.ac;
        uint32_t e = lut[table + (bits >> (32 - kLutK))];
        if (lut_esc(e)) {
            const uint32_t n = lut_esc_bits(e);
            e = lut[table + (uint32_t)kLutL1 + lut_esc_offset(e) + ((bits >> (32 - kLutK - n)) & ((1u << n) - 1u))];
        }
        s.size = lut_size(e);
        s.slots = lut_adv(e);
        s.coded = s.is_dc ? s.slots == 1u : s.slots != 0u;
        s.value = symbol_value(bits, lut_total(e), s.size);
        l.p += lut_total(e);
        l.z += s.slots;
        s.done = l.z >= 64u;
        if (s.done) {
            l.z = 0u;
            l.u = l.u + 1u == upm ? 0u : l.u + 1u;
            ++l.nb;
        }
        ++symbols;
        return s;
    }
    // behind a symbol: in the padding in front of the interval that starts at B, or past its start
    void enter_interval(PlainLane& l, uint32_t B) {
        const uint32_t left = B - l.p;
        if (B == kNoBoundary || (l.p < B && (left > 7u || (~peek(l.p) >> (32u - left)) != 0u))) return;
        l.p = B;
        l.u = l.z = 0u;
    }

    // Synchronisation pass: symbols that start before `limit`.
    void sync(PlainLane& l, uint32_t limit, int64_t& dc) {
        while (l.p < limit) {
            const Symbol s = next(l);
            if (s.is_dc) dc += (int64_t)s.value * ((int64_t)1 << (15u * units[s.u].comp));
        }
    }
    template <class BWord>
    void sync_rst(PlainLane& l, uint32_t limit, int64_t& dc, uint32_t& crossed, BWord bword) {
        uint32_t B = next_boundary(l.p, limit + 64u, bword);
        while (l.p < limit) {
            if (l.p == B) {  // the symbol that starts an interval
                dc = 0;
                crossed = 1u;
                B = next_boundary(B + 1u, limit + 64u, bword);
            }
            sync(l, l.p + 1u, dc);
            enter_interval(l, B);
        }
    }

    // Write pass: store(unit, index, value) for every coefficient and DC value; `flags` collects kSt* bits.
    template <class Store>
    void write_one(PlainLane& l, uint32_t& unit, int32_t pred[3], Store store, uint32_t& flags) {
        const Symbol s = next(l);
        if (s.is_dc && s.coded) store(unit, 0u, (int16_t)(pred[units[s.u].comp] += s.value));
        if (!s.is_dc && s.size != 0u && s.z + s.slots <= 64u) store(unit, s.z + s.slots - 1u, (int16_t)s.value);
        if (!s.coded || (!s.is_dc && s.slots != kAdvEob && s.z + s.slots > 64u)) flags |= kStInvalid;
        unit += s.done ? 1u : 0u;
    }
    template <class Store>
    void write(PlainLane& l, uint32_t limit, uint32_t& unit, uint32_t total, int32_t pred[3], Store store, uint32_t& flags) {
        while (l.p < limit && unit < total) write_one(l, unit, pred, store, flags);
    }
    template <class Store, class BWord>
    void write_rst(PlainLane& l, uint32_t limit, uint32_t& unit, uint32_t total, uint32_t units_per_interval, int32_t pred[3], Store store,
                   uint32_t& flags, BWord bword) {
        uint32_t B = next_boundary(l.p, limit + 64u, bword);
        while (l.p < limit && unit < total) {
            if (l.p == B) {
                pred[0] = pred[1] = pred[2] = 0;
                if (unit % units_per_interval != 0u) flags |= kStInvalid;
                B = next_boundary(B + 1u, limit + 64u, bword);
            }
            write_one(l, unit, pred, store, flags);
            enter_interval(l, B);
        }
    }
};
template <class Peek>
PlainScan<Peek> plain_scan(const PlainUnit* units, uint32_t upm, const uint16_t* lut, Peek peek) {
    return PlainScan<Peek>{units, upm, lut, peek};
}

}  // namespace jpgd
