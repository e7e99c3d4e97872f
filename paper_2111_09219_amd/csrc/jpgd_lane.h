// What one lane does: decode JPEG syntax elements from an arbitrary bit position and decoder state
// (paper, Algorithm 2 "decode_subsequence" and the function decode_next_symbol it calls).
// Host/device code.  The lanes' inner loops (sync_span, write_span) are written out in assembly in jpgd_kernels.h; what stands
// here says what every value in them is, and is what the tests of the CPU-only run hold to plain decoders.  Everything
// else - how the tables are laid out, how a lane starts, restart intervals, chunks of coefficients - is what the kernels inline.
//
// One symbol depends on the previous one through a short chain: table entry -> code and value length -> shifted window -> next
// table index -> LDS read.  A lone wavefront spends most of its time on that chain, so the entry of the next symbol is asked
// for as soon as the one in hand has been taken apart, and everything else (DC sums, unit bookkeeping, stores, stream words) is
// done while that read is in flight.  A codeword longer than the first-level index is resolved as a step of its own that
// takes no bits, so the common path has no second dependent read.
//
// Decoder state of the paper, (p, n, c, z): c is refined to the data unit inside the MCU (two decoders inside different
// luminance units of a 4:2:0 MCU agree on the component but not on what follows) and n kept as completed data units (see
// SInfo).
#pragma once
#include "jpgd_common.h"

namespace jpgd {

// The value bits are the last `size` of the `total` bits a symbol takes; "signed ones' complement" (paper,
// Section 2): a leading 1 means the bits are the value itself, a leading 0 means value = bits - (2^size - 1);
// size 0 gives 0.  peek holds the symbol from its most significant bit on.  With the field read as a signed
// number s (leading 1 = negative): value = s + 2^size if s < 0, else s - 2^size + 1.
JPGD_HD int32_t value_of_field(int32_t s, uint32_t size) {
    // s + 2^size if s < 0, s - (2^size - 1) otherwise: subtract 2^size - 1 with all its bits flipped in the first case
    return s - (int32_t)(((1u << size) - 1u) ^ (uint32_t)(s >> 31));
}
JPGD_HD int32_t symbol_value(uint32_t peek, uint32_t total, uint32_t size) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int32_t s = __builtin_amdgcn_sbfe((int32_t)peek, (32u - total) & 31u, size);
#else
    const uint32_t raw = (peek >> ((32u - total) & 31u)) & ((1u << size) - 1u);
    const int32_t s = size ? (int32_t)(raw << (32u - size)) >> (32u - size) : 0;
#endif
    return value_of_field(s, size);
}

// DC-difference sums of the three components, kept in one 64-bit accumulator with 15-bit fields
// (component c at bit 15*c) so that a single multiply-add updates the right one.  A subsequence's
// true sums are differences of two quantised DC values and fit easily; sums of lanes that are not
// synchronised may spill into the neighbouring field, and are discarded anyway.
JPGD_HD void dc_unpack(int64_t acc, int32_t& d0, int32_t& d1, int32_t& d2) {
    d0 = (int32_t)((int64_t)((uint64_t)acc << 49) >> 49);
    acc = (acc - d0) >> 15;
    d1 = (int32_t)((int64_t)((uint64_t)acc << 49) >> 49);
    acc = (acc - d1) >> 15;
    d2 = (int32_t)acc;
}

// ---- the lanes of the synchronisation pass -----------------------------------------------------------------
// write = false in Algorithm 2: state, count of completed units and sums of DC differences, on tables laid out for it in LDS.  A
// 32-bit entry per first-level index says at once what its symbol takes, what the symbol behind it takes where the index
// holds that one's whole codeword too (build_pairs), and how many value bits a DC symbol has.  Position and zig-zag index
// are one register that an entry is added to.
// The pass needs no coefficients, so one step may take two symbols: the second only behind an AC symbol that leaves its unit
// open (it belongs to the same unit and table then), and only where it starts before the end of the subsequence, like any
// other.  Such a step is exactly two steps of one symbol.
//
// What bounds it: a lane's next look-up waits for the one before (about 130 cycles of LDS), and behind that for the
// instructions between an entry's arrival and the next request, 4 cycles each; with several wavefronts on a SIMD, for
// all instructions of a step.  So the words on the way from entry to request are kept few, everything else stands behind
// the request, and an escape (a codeword longer than the index) is followed up without a branch, which would cost a
// lone wavefront more than the instructions it skips: 46 vector instructions and three LDS reads a step.  On the 16-bit
// entries of build_lut with pair bytes beside them a step took 62 and five, two thirds of them in front of the request.
// Measured, on those / on these (kernels, us): 15360x8640 first kernel 697 / 611, second 890 / 848; 256 images of
// 512x384 240 / 213; 24 images of 2047x1535 337 / 305; one 1001x667 image 104 / 89; 3001x2003 with an interval per MCU row
// (single symbols before) 122 / 97.
//
//   entry, bits 0..4   bits the symbol takes
//          bits 9..14  zig-zag slots it covers
//          bit  15     set, with bit 31, in an escape: bits 0..4 and 9..14 are zero, bits 6..8 = n, bits 18..30 = 8-byte
//                      word of the tables from which on the subtable lies that the n bits from the last bit of a 10-bit
//                      index on point into
//          bits 16..19 bits that the symbol behind it takes, bits 25..30 the slots that one covers (0: no second symbol;
//                      an end of block covers kAdvEob like any other)
//          bits 20..23 DC tables: value bits of the symbol
// The write pass's tables differ in that nothing is said of a second symbol: bits 20..23 are the value bits of an AC
// symbol too, bit 16 is set for coefficients and runs of sixteen zeros, which must not reach past the end of the unit,
// bit 17 where no codeword starts, bit 30 where there is a value to be stored and bit 29 beside it for DC symbols (as signed
// numbers: from kWriteValue on a value, from kWriteDc on a DC value, escapes below zero).
constexpr uint32_t kSyncDcK = 9u;              // bits of a first-level index: DC tables (half the size; their codes are short),
constexpr uint32_t kSyncAcK = (uint32_t)kLutK; // AC tables
constexpr uint32_t kSyncDcBytes = 4u << kSyncDcK, kSyncAcBytes = 4u << kSyncAcK;
constexpr uint32_t kSyncEsc = 0x8000u;         // also: the carry out of the zig-zag index, "data unit complete"
constexpr uint32_t kSyncStep = 0x7E1Fu;        // position and slots
constexpr uint32_t kSyncSecond = 0x7E0Fu;      // the same of the second symbol, in the upper half
constexpr uint32_t kSyncPairBits = 9u;         // most bits a first symbol with a second one behind it takes
static_assert(kSyncDcK == kSyncAcK - 1u, "subtables of both kinds are indexed from the last bit of a 10-bit index on");

// second-level entry (or first-level one that is no escape) of build_lut, with pair byte pb (0: none)
JPGD_HD uint32_t sync_entry(uint32_t e, bool is_dc, uint32_t pb) {
    const uint32_t slots = pb >> 4;
    return (e & kSyncStep) | (is_dc ? lut_size(e) << 20 : ((pb & 15u) | ((slots == 15u ? kAdvEob : slots) << 9)) << 16);
}
constexpr uint32_t kWriteInside = 1u << 16, kWriteNoCode = 1u << 17;
constexpr int32_t kWriteValue = 1 << 30, kWriteDc = 3 << 29;
JPGD_HD uint32_t write_entry(uint32_t e, bool is_dc) {
    const uint32_t slots = lut_adv(e), size = lut_size(e);
    const bool coded = is_dc ? slots == 1u : slots != 0u;
    return (e & kSyncStep) | (size << 20) | (!coded ? kWriteNoCode : !is_dc && slots != kAdvEob ? kWriteInside : 0u) |
           (uint32_t)(!coded ? 0 : is_dc ? kWriteDc : size != 0u ? kWriteValue : 0);
}
// either, as the tables of the pass need it
template <bool WRITE>
JPGD_HD uint32_t pass_entry(uint32_t e, bool is_dc, uint32_t pb) { return WRITE ? write_entry(e, is_dc) : sync_entry(e, is_dc, pb); }
// escape into a subtable indexed by n bits, from byte `at` of the tables on (a multiple of 8)
JPGD_HD uint32_t sync_escape(uint32_t n, uint32_t at) { return 0x80000000u | kSyncEsc | (n << 6) | ((at >> 3) << 18); }
// byte of the tables at which the entry lies that escape e leads to
JPGD_HD uint32_t sync_escape_at(uint32_t e, uint32_t peek) {
    const uint32_t n = (e >> 6) & 7u;
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t i = __builtin_amdgcn_ubfe(peek, 23u - n, n);
#else
    const uint32_t i = (peek >> (23u - n)) & ((1u << n) - 1u);
#endif
    return ((e >> 15) & 0xFFF8u) + (i << 2);
}
// first-level entry i of an AC table; l2: byte of the tables from which on the table's second level lies, entry by entry
template <bool WRITE = false>
JPGD_HD uint32_t sync_ac_entry(uint32_t i, uint32_t e, uint32_t pb, uint32_t l2) {
    if (!lut_esc(e)) return pass_entry<WRITE>(e, false, pb);
    const uint32_t n = lut_esc_bits(e);
    return sync_escape(n + 1u, l2 + 4u * lut_esc_offset(e) - (n ? (i & 1u) << (n + 2u) : 0u));
}
// Entry i of a DC table from entries 2i and 2i+1 of build_lut's: n such that they need a subtable of 2^(n+1) entries, or
// 0xFFFFFFFF if both are the same symbol (or no codeword).
JPGD_HD uint32_t sync_dc_sub(uint32_t a, uint32_t b) {
    if (a == b && !(lut_esc(a) && lut_esc_bits(a) != 0u)) return 0xFFFFFFFFu;
    const uint32_t na = lut_esc(a) ? lut_esc_bits(a) : 0u, nb = lut_esc(b) ? lut_esc_bits(b) : 0u;
    return na > nb ? na : nb;
}
// entry j of that subtable; l2: second level of build_lut's table.  (An escape without further bits stands for "no
// codeword", the first entry there.)
template <bool WRITE = false, class L2>
JPGD_HD uint32_t sync_dc_sub_entry(uint32_t a, uint32_t b, uint32_t n, uint32_t j, L2 l2) {
    const uint32_t e = j >> n ? b : a;
    if (!lut_esc(e)) return pass_entry<WRITE>(e, true, 0u);
    const uint32_t k = lut_esc_bits(e);
    return pass_entry<WRITE>(l2[lut_esc_offset(e) + ((j & ((1u << n) - 1u)) >> (n - k))], true, 0u);
}
template <bool WRITE = false>
JPGD_HD uint32_t sync_dc_direct(uint32_t a) { return pass_entry<WRITE>(lut_esc(a) ? kDcNoCode : a, true, 0u); }

// Words of subtables that a table of build_lut needs in this layout (at most 1022).
inline uint32_t sync_sub_words(const uint16_t* lut, bool is_dc) {
    uint32_t words = 0u;
    if (is_dc) {
        for (uint32_t i = 0; i < (uint32_t)kLutL1; i += 2u) {
            const uint32_t n = sync_dc_sub(lut[i], lut[i + 1u]);
            if (n != 0xFFFFFFFFu) words += 2u << n;
        }
        return words;
    }
    words = 2u;
    for (uint32_t i = 0; i < (uint32_t)kLutL1; ++i)
        if (lut_esc(lut[i])) {
            const uint32_t end = lut_esc_offset(lut[i]) + (1u << lut_esc_bits(lut[i]));
            if (end > words) words = end;
        }
    return (words + 1u) & ~1u;
}

// One row per data unit of the MCU: bytes of the tables at which its AC table and the next unit's DC table start, the
// factor of its component in the DC sums, and the byte of the rows at which the next unit's row lies.
struct alignas(16) SyncRow {
    uint32_t ac, dc_next, dcmul, next;
};

// A lane between two symbols.  The window is two words and the offset of the next bit in them, 1 to 32 (so that one
// funnel shift by 0 to 31 gives the next 32 bits); S holds the offset less one in bits 0..4 and the zig-zag index in bits
// 9..14.
struct SyncLane {
    uint32_t S;
    uint32_t row;        // byte of the current unit's row, in the bytes of the Row functor
    uint32_t e;          // entry of the symbol that comes next, already asked for
    uint32_t hi, lo, ahead;
    uint32_t at;         // bit at which `ahead` starts, in the bits of the Word functor
    uint32_t nb;         // data units completed since it was last cleared
};

JPGD_HD uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t s) {  // by s & 31 to the right
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_alignbit(hi, lo, s);
#else
    return (uint32_t)(((((uint64_t)hi) << 32) | lo) >> (s & 31u));
#endif
}
// position of the next bit, less one, plus 64 (the two words before `at`)
JPGD_HD uint32_t sync_at(const SyncLane& l) { return (l.S & 31u) | l.at; }
constexpr uint32_t kSyncBias = 63u;
JPGD_HD uint32_t sync_pos(const SyncLane& l) { return sync_at(l) - kSyncBias; }

JPGD_HD uint32_t sync_peek(const SyncLane& l) { return funnel(l.hi, l.lo, ~l.S); }

// word(b): the stream word that starts at bit b (a multiple of 32); tab(k): 32-bit entry at byte k of the tables; rows(k):
// the SyncRow at byte k; the rows of the upm units lie from byte row0 on.  p: bit to start at, in the bits of `word`; z, u:
// zig-zag index and data unit.
template <class Word, class Tab, class Row>
JPGD_HD void sync_start(SyncLane& l, uint32_t p, uint32_t u, uint32_t z, uint32_t upm, uint32_t row0, Word word, Tab tab, Row rows) {
    const uint32_t w = (p + 31u) & ~31u;
    l.hi = (p & 31u) ? word(w - 32u) : 0u;  // (at the first bit of a word the offset is 32: nothing of it is used)
    l.lo = word(w);
    l.ahead = word(w + 32u);
    l.at = w + 32u;
    l.S = ((p + 31u) & 31u) | (z << 9);
    l.row = row0 + u * (uint32_t)sizeof(SyncRow);
    const uint32_t dc = rows(row0 + ((u ? u : upm) - 1u) * (uint32_t)sizeof(SyncRow)).dc_next;
    const uint32_t peek = sync_peek(l);
    l.e = tab(z == 0u ? dc + ((peek >> (32u - kSyncDcK)) << 2) : rows(l.row).ac + ((peek >> (32u - kSyncAcK)) << 2));
}

// Decodes while the next symbol starts before bit `limit` (of `word`).  A second symbol is left to the next step where
// it might start behind `limit`.
template <class Word, class Tab, class Row>
JPGD_HD void sync_span(SyncLane& l, uint32_t limit, int64_t& dcacc, Word word, Tab tab, Row rows) {
    const uint32_t stop = limit + kSyncBias, last_pair = stop - kSyncPairBits;
    uint32_t pos = sync_at(l);
    if (pos >= stop) return;
    uint32_t peek = sync_peek(l);
    SyncRow row = rows(l.row);
#if defined(__HIP_DEVICE_COMPILE__)
    // (Keeps the compiler from merging this read with the one at the end of a step into one at the top of the loop, where
    // every step would wait for it.)
    asm volatile("" : "+v"(row.ac), "+v"(row.dc_next), "+v"(row.dcmul), "+v"(row.next));
#endif
    do {
        const bool late = pos >= last_pair;
        const uint32_t e = l.e, before = peek;
        const bool esc = (int32_t)e < 0;
        const uint32_t s1 = l.S + (e & 0xFFFFu);
        const bool one = late || s1 >= kSyncEsc;  // (an escape has no second symbol either)
        const uint32_t s2 = s1 + (one ? 0u : (e >> 16) & kSyncSecond);
        const bool ends = s2 >= kSyncEsc;         // the unit is complete, or an escape
        const uint32_t word_on = s2 & 32u;
        l.hi = word_on ? l.lo : l.hi;
        l.lo = word_on ? l.ahead : l.lo;
        peek = funnel(l.hi, l.lo, ~s2);
        const uint32_t next = (ends ? row.dc_next : row.ac) + ((peek >> (ends ? 32u - kSyncDcK : 32u - kSyncAcK)) << 2);
        const uint32_t sub = sync_escape_at(e, peek);
        uint32_t size = (e >> 20) & 15u, total = e & 31u;
#if defined(__HIP_DEVICE_COMPILE__)
        total = 0u - e;  // (the offset of the value's bits, taken modulo 32)
        asm volatile("" : "+v"(size), "+v"(total));  // (the entry's register is free for the next one from here on)
#endif
        l.e = tab(esc ? sub : next);
        l.at += word_on;
        l.ahead = word(l.at);
        const bool done = ends && !esc;
        l.S = s2 & (done ? 31u : kSyncStep);
        l.nb += done ? 1u : 0u;
        l.row = done ? row.next : l.row;
        pos = sync_at(l);
        // value of a DC symbol (0 with the 0 value bits that every other entry has)
        const int32_t mul = (int32_t)(esc ? 0u : row.dcmul);
        row = rows(l.row);
#if defined(__HIP_DEVICE_COMPILE__)
        const int32_t v = value_of_field(__builtin_amdgcn_sbfe((int32_t)before, total, size), size);
#else
        const int32_t v = symbol_value(before, total, size);
#endif
        dcacc += (int64_t)v * (int64_t)mul;
    } while (pos < stop);
}

// ---- the lanes of the write pass ---------------------------------------------------------------------------
// The same walk, one symbol per step (write = true in Algorithm 2), on tables in the same layout: every non-zero coefficient
// goes to 64*unit + zig-zag index, DC values un-differenced.  Without branches except around the store itself: a
// wavefront holds lanes in every kind of symbol at once, so each arm of a branch would be walked anyway.
// What bounds it is the length of a step in a wavefront that has its SIMD nearly to itself: 680 cycles on the 4096x4096
// image where the stores are scattered over 64 lines, 450 of them without any store (the kernels' assembly, 400 with it:
// write_span_device); a loop for the zeros between two values, for stretches of dense units, was 100 more and is gone since
// the coefficients are always cleared first.
// Kernel before / now, cleared ahead (us): 24 images of 2047x1535 104 / 82, 4963x7013 gray 31 / 21, 1001x667 28 / 23, one
// 1600x1200 image 46 / 38, 3001x2003 41 / 36; 15360x8640 (cleared here) 412 / 384.
// The predictors are kept in the order in which the components come next: the current unit's in p0, so that a DC symbol need
// not choose; they move up where the component changes (`dcmul` of a write pass's row: 1 if the unit behind it is of another
// component, else 0).
struct WriteLane {
    SyncLane s;
    SyncRow row;         // the current unit's
    uint32_t peek;
    uint32_t unit;       // index of the data unit being decoded
    int32_t p0, p1, p2;
    uint32_t seen;       // bit 16: a symbol ran past the end of its unit; bit 17: bits that start no codeword
};
constexpr uint32_t kWriteBad = 3u << 16;
// the predictors of components 0, 1 and 2 in the order for a unit of component comp
JPGD_HD void write_predictors(WriteLane& l, uint32_t comp, int32_t d0, int32_t d1, int32_t d2) {
    l.p0 = comp == 0u ? d0 : comp == 1u ? d1 : d2;
    l.p1 = comp == 0u ? d1 : comp == 1u ? d2 : d0;
    l.p2 = comp == 0u ? d2 : comp == 1u ? d0 : d1;
}
template <class Word, class Tab, class Row>
JPGD_HD void write_start(WriteLane& l, uint32_t p, uint32_t u, uint32_t z, uint32_t upm, uint32_t row0, Word word, Tab tab, Row rows) {
    sync_start(l.s, p, u, z, upm, row0, word, tab, rows);
    l.row = rows(l.s.row);
    l.peek = sync_peek(l.s);
}
template <class Word, class Tab, class Row, class Store>
JPGD_HD void write_step(WriteLane& l, Word word, Tab tab, Row rows, Store store) {
    const uint32_t e = l.s.e, before = l.peek;
    const bool esc = (int32_t)e < 0;
    const bool dc = (int32_t)e >= kWriteDc, valued = (int32_t)e >= kWriteValue;
    const uint32_t s2 = l.s.S + (e & 0xFFFFu);
    const bool ends = s2 >= kSyncEsc;  // the unit is complete, or an escape
    const uint32_t word_on = s2 & 32u;
    l.s.hi = word_on ? l.s.lo : l.s.hi;
    l.s.lo = word_on ? l.s.ahead : l.s.lo;
    l.peek = funnel(l.s.hi, l.s.lo, ~s2);
    const uint32_t next = (ends ? l.row.dc_next : l.row.ac) + ((l.peek >> (ends ? 32u - kSyncDcK : 32u - kSyncAcK)) << 2);
    const uint32_t sub = sync_escape_at(e, l.peek);
    uint32_t size = (e >> 20) & 15u, total = e & 31u;
    // (bit 16 of the sum is set from 65 slots on, bit 17 always)
    l.seen |= e & (s2 + (kWriteNoCode + kWriteInside - (65u << 9)));
#if defined(__HIP_DEVICE_COMPILE__)
    total = 0u - e;  // (the offset of the value's bits, taken modulo 32)
    asm volatile("" : "+v"(size), "+v"(total), "+v"(l.seen));  // (the entry's register is free for the next one from here on)
#endif
    l.s.e = tab(esc ? sub : next);
    l.s.at += word_on;
    l.s.ahead = word(l.s.at);
    const bool done = ends && !esc;
    l.s.S = s2 & (done ? 31u : kSyncStep);
    l.s.row = done ? l.row.next : l.s.row;
    const bool other = done && l.row.dcmul != 0u;
    l.row = rows(l.s.row);
#if defined(__HIP_DEVICE_COMPILE__)
    const int32_t v = value_of_field(__builtin_amdgcn_sbfe((int32_t)before, total, size), size);
#else
    const int32_t v = symbol_value(before, total, size);
#endif
    l.p0 += dc ? v : 0;
    // where the symbol ends: a coefficient sits in the last slot it covers (after its run of zeros); a DC symbol, which
    // yields the predictor without value bits too, in slot 0
    if (valued && s2 < (65u << 9)) store(l.unit, (s2 >> 9) - 1u, (int16_t)(dc ? l.p0 : v));
    const int32_t q = l.p0;
    l.p0 = other ? l.p1 : l.p0;
    l.p1 = other ? l.p2 : l.p1;
    l.p2 = other ? q : l.p2;
    l.unit += done ? 1u : 0u;
}

// Decodes while the next symbol starts before bit `limit` (of `word`), up to the image's last data unit.
template <class Word, class Tab, class Row, class Store>
JPGD_HD void write_span(WriteLane& l, uint32_t limit, uint32_t total_units, Word word, Tab tab, Row rows, Store store) {
    const uint32_t stop = limit + kSyncBias;
    while (sync_at(l.s) < stop && l.unit < total_units) write_step(l, word, tab, rows, store);
}

// Coefficients leave a lane four at a time.  Every value as a store of its own makes 64 two-byte requests per dense data unit,
// and the number of requests, not of bytes, is what the memory system charges for: the values of four neighbouring slots (one
// aligned 8-byte chunk of the output) are gathered in a register pair and stored together when the lane moves on to another
// chunk.  The zeros among them are the lane's own (the chunk lies inside the range of slots this lane covers), except in the
// chunk the lane starts in, if it starts in the middle of one, and in the chunk it ends in: those are shared with the
// neighbouring lanes and get their values one by one, when the lane is done.  (Measured too: eight slots per store, no faster
// on dense units, slower on sparse ones; chunks counted from the lane's first slot on, whose first one is nobody else's but
// which lie across 8-byte words, 48 frames of 1920x1088 4:4:4 in 499 us a call against 476.)
struct WriteChunk {
    uint64_t acc;     // chunk being gathered
    uint32_t cur;     // its first slot
    uint32_t shared;  // first slot of the chunk the lane starts in, if a neighbour holds its start, else 0xFFFFFFFF
    uint64_t first;   // what was gathered in that one
};
JPGD_HD WriteChunk chunk_start(uint32_t slot) {
    const uint32_t cur = slot & ~3u;
    return WriteChunk{0ull, cur, (slot & 3u) ? cur : 0xFFFFFFFFu, 0ull};
}
// the lane moves on to a later chunk: the one it leaves reaches up to its end inside the lane's range (a chunk left without a
// value costs a store of zeros onto the cleared background, once per lane at most)
template <class Store8>
JPGD_HD void chunk_value(WriteChunk& c, uint32_t slot, int16_t v, Store8 store8) {
    const uint32_t chunk = slot & ~3u;
    if (chunk != c.cur) {
        if (c.cur != c.shared) store8(c.cur, c.acc);
        else c.first = c.acc;
        c.acc = 0ull;
        c.cur = chunk;
    }
    c.acc |= (uint64_t)(uint16_t)v << ((slot & 3u) * 16u);
}
// the chunks shared with neighbouring lanes, onto the cleared background
template <class Store1>
JPGD_HD void chunk_ends(const WriteChunk& c, Store1 store1) {
    for (uint32_t k = 0; k < 4u; ++k) {
        const int16_t v = (int16_t)(uint16_t)(c.acc >> (16u * k)), w = (int16_t)(uint16_t)(c.first >> (16u * k));
        if (v != 0) store1(c.cur + k, v);
        if (w != 0) store1(c.shared + k, w);
    }
}

// ---- the walk of a whole wavefront ---------------------------------------------------------------------------
// What the walk through a single chain (coop_span_sync in jpgd_kernels.h) needs to know of the image's data units.
//
// Data units that share a DC and an AC table are of one kind; with a pair of tables per component there are at most three.
// The word, made by the host: bits 0..11 kind of each unit of the MCU (2 bits each), from kWalkSlots on the slots of the DC
// and the AC table of kinds 0, 1 and 2 (3 bits each; those of a kind that is not there are kind 0's), bit kWalkThree: there
// are three.
constexpr uint32_t kWalkSlots = 12u, kWalkThree = 30u;
JPGD_HD uint32_t walk_word(uint32_t upm, uint32_t sched_dc, uint32_t sched_ac) {
    uint32_t word = 0u, kinds = 0u, slots[3] = {0u, 0u, 0u};
    for (uint32_t u = 0; u < upm; ++u) {
        const uint32_t mine = ((sched_dc >> (4u * u)) & 15u) | ((sched_ac >> (4u * u)) & 15u) << 3;
        uint32_t k = 0;
        while (k < kinds && slots[k] != mine) ++k;
        if (k == kinds) slots[kinds++] = mine;
        word |= k << (2u * u);
    }
    for (uint32_t k = 0; k < 3u; ++k) word |= slots[k < kinds ? k : 0u] << (kWalkSlots + 6u * k);
    return word | (kinds == 3u ? 1u << kWalkThree : 0u);
}

// Data unit u of the MCU for the walk: index of the unit that follows (bits 0..3), its kind (4..5), and where its DC
// differences go in the walk's two sums: shift inside the first word (10..14: 0 for component 0, 16 for component 1), or the
// second word (bit 15, component 2)
constexpr uint32_t kUwKind = 4u, kUwShift = 10u, kUwSecond = 15u;
JPGD_HD uint32_t walk_unit(uint32_t walk, uint32_t sched_comp, uint32_t upm, uint32_t u) {
    const uint32_t next = u + 1u == upm ? 0u : u + 1u, comp = (sched_comp >> (4u * u)) & 15u;
    return next | (((walk >> (2u * u)) & 3u) << kUwKind) | (comp == 2u ? 1u << kUwSecond : comp * 16u << kUwShift);
}

// Where the tables of kind k lie; tab: byte at which the tables begin.
JPGD_HD uint32_t walk_dc(uint32_t walk, uint32_t k, uint32_t tab) { return tab + ((walk >> (kWalkSlots + 6u * k)) & 7u) * kSyncDcBytes; }
JPGD_HD uint32_t walk_ac(uint32_t walk, uint32_t k, uint32_t ndc, uint32_t tab) {
    return tab + ndc * kSyncDcBytes + (((walk >> (kWalkSlots + 6u * k + 3u)) & 7u) - ndc) * kSyncAcBytes;
}

// ---- restart intervals -------------------------------------------------------------------------------
// A scan with restart intervals (DRI) is a chain of independently coded intervals: each ends with up to seven
// 1-bits of padding and a marker RSTm, and the next starts byte-aligned with the DC predictors at zero.  The
// unstuff kernels drop the markers and mark the first byte of every interval in a bitmap (one bit per byte
// of the unstuffed stream; bit b of word k stands for byte 32k + b).  The paper does not treat restart
// markers.  The rules below are stated on positions alone, so that a decoder in any state obeys them, and on
// the synchronised chain they are what a sequential decoder does:
//   * after a symbol, if the next interval starts at most 7 bits further on and those bits are all 1, or if
//     the symbol ran past that start, the decoder moves to the start with z = 0 and u = 0 (a real symbol
//     never consists of 1-bits only: the all-ones codeword is reserved);
//   * a symbol that starts at the first bit of an interval finds the DC sums / predictors at zero.
// Every decoder is therefore synchronised from the next interval on, whatever it did before.

constexpr uint32_t kNoBoundary = 0xFFFFFFFFu;

// first bit position B >= from_bit, B < end_bit, at which an interval starts; bword(k) = word k of the bitmap
template <class BWord>
JPGD_HD uint32_t next_boundary(uint32_t from_bit, uint32_t end_bit, BWord bword) {
    const uint32_t byte = (from_bit + 7u) >> 3, endb = (end_bit + 7u) >> 3;
    if (byte >= endb) return kNoBoundary;
    uint32_t k = byte >> 5;
    uint32_t m = bword(k) & (0xFFFFFFFFu << (byte & 31u));
    for (;;) {
        if (m) {
            const uint32_t b = (k << 5) + (uint32_t)__builtin_ctz(m);
            return b < endb ? b << 3 : kNoBoundary;
        }
        ++k;
        if ((k << 5) >= endb) return kNoBoundary;
        m = bword(k);
    }
}

// Synchronisation pass over a stream with restart intervals.  `crossed` is set when a symbol of this span started an interval
// (dcacc then holds the sums since the last such symbol).  Boundaries are positions in the image's stream: a position there
// plus `org` is a bit of `word`.  start(p): sync_start at bit p with u = z = 0; span(limit): sync_span.
// A fast loop up to the neighbourhood of the next interval start, then a careful one of single symbols.  (The single loop of
// the write pass below was measured here too: the overflow rounds are a chain of dependent symbols in a lone wavefront, and
// the extra tests per symbol cost them more -- 4096x4096 with one interval per MCU row: 0.93 against 0.78 ms -- than walking
// a span twice costs the few wavefronts that meet an interval start.)
template <class Start, class Span, class BWord>
JPGD_HD void sync_span_rst(SyncLane& l, uint32_t limit, int64_t& dcacc, uint32_t& crossed, uint32_t org, Start start, Span span,
                           BWord bword) {
    const uint32_t end = limit - org;
    uint32_t from = sync_pos(l) - org;
    for (;;) {
        const uint32_t B = next_boundary(from, end + 64u, bword);
        // a symbol that starts 40 bits before B ends more than 7 bits before it
        uint32_t calm = end;
        if (B != kNoBoundary && B < end + 39u) calm = B >= 39u ? B - 39u : 0u;
        if (from < calm) span(calm + org);
        if (B == kNoBoundary) break;
        uint32_t pos = sync_pos(l) - org;
        bool next_interval = false;
        while (pos < end) {
            if (pos == B) {  // this symbol starts the interval
                dcacc = 0;
                crossed = 1u;
                from = B + 1u;
                next_interval = true;
                break;
            }
            span(pos + org + 1u);  // one symbol
            pos = sync_pos(l) - org;
            const uint32_t r = B - pos;
            if (pos >= B || (r <= 7u && (~sync_peek(l) >> (32u - r)) == 0u)) {
                start(B + org);
                pos = B;
            }
        }
        if (!next_interval) break;
    }
}

// Write pass over a stream with restart intervals: the predictors return to zero where an interval starts.  `org` as in
// sync_span_rst.  An interval holds units_per_interval data units (all but the last of the scan): a start reached at any
// other unit count means damaged data and is flagged (kStInvalid in *flags).
// One loop for all lanes: a lane near an interval start does its checks before and after the same write_step the others
// execute.  With a fast loop and a careful loop one after the other, a wavefront in which a few lanes meet an interval
// start walks its span up to three times (the fast loop for the others, the careful one, the fast one again for what
// follows the start); the write kernel, whose wavefronts all have full spans to decode, is a third faster this way on
// streams with one interval per MCU row.
template <class Word, class Tab, class Row, class Store, class BWord>
JPGD_HD void write_span_rst(WriteLane& l, uint32_t limit, uint32_t total_units, uint32_t units_per_interval, uint32_t org,
                            uint32_t upm, uint32_t row0, Word word, Tab tab, Row rows, Store store, BWord bword, uint32_t* flags) {
    const uint32_t end = limit - org;
    auto calm_until = [&](uint32_t B) { return B != kNoBoundary && B < end + 39u ? (B >= 39u ? B - 39u : 0u) : end; };
    uint32_t pos = sync_pos(l.s) - org;
    uint32_t B = next_boundary(pos, end + 64u, bword);
    uint32_t calm = calm_until(B);
    while (l.unit < total_units) {
        const bool near = pos >= calm;
        if (near) {
            if (B == kNoBoundary || pos >= end) break;
            if (pos == B) {
                l.p0 = l.p1 = l.p2 = 0;
                if (l.unit % units_per_interval != 0u) *flags |= kStInvalid;
                B = next_boundary(B + 1u, end + 64u, bword);
                calm = calm_until(B);
                continue;
            }
        }
        write_step(l, word, tab, rows, store);
        pos = sync_pos(l.s) - org;
        if (near && (pos >= B || (B - pos <= 7u && (~l.peek >> (32u - (B - pos))) == 0u))) {
            write_start(l, B + org, 0u, 0u, upm, row0, word, tab, rows);
            pos = B;
        }
    }
}

}  // namespace jpgd
