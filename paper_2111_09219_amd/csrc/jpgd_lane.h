// What one lane does: decode JPEG syntax elements from an arbitrary bit position and decoder state
// (paper, Algorithm 2 "decode_subsequence" and the function decode_next_symbol it calls).
// Host/device code: the kernels inline it, and a host build of the same functions is exercised
// on the CPU by the test suite.
//
// The loop is software-pipelined by hand.  One symbol depends on the previous one through a short
// chain -- table entry -> code + value length -> shifted window -> next table index -> LDS read -- and a
// lone wavefront spends most of its time waiting on that chain.  So the table entry of the NEXT
// symbol is requested as soon as the current entry has been unpacked, and everything that is not on
// the chain (DC sums, unit bookkeeping, stores, fetching stream words) is done while that read is in
// flight.  A codeword longer than the first-level index is resolved as an iteration of its own that
// consumes no bits, so the common path has no second dependent read.
#pragma once
#include "jpgd_common.h"

namespace jpgd {

// What a lane needs to know about one data unit of the MCU: where the tables of its symbols are, which
// DC sum it feeds, and which unit follows.  One row per data unit, 16 bytes, read as a whole.
struct alignas(16) UnitRow {
    uint32_t tb_ac;       // first entry of the unit's AC table inside the LUT array
    uint32_t tb_dc_next;  // first entry of the DC table of the unit that follows
    uint32_t dcmul;       // 1 << (15 * component): the component's field of the packed DC sums
    uint32_t next;        // index of the unit that follows
};

// sched_*: 4 bits per data unit (see ImgDesc)
JPGD_HD UnitRow make_unit_row(uint32_t u, uint32_t upm, uint32_t sched_dc, uint32_t sched_ac, uint32_t sched_comp) {
    UnitRow r;
    const uint32_t un = u + 1u == upm ? 0u : u + 1u;
    r.tb_ac = ((sched_ac >> (4u * u)) & 15u) * (uint32_t)kLutEntries;
    r.tb_dc_next = ((sched_dc >> (4u * un)) & 15u) * (uint32_t)kLutEntries;
    r.dcmul = 1u << (15u * ((sched_comp >> (4u * u)) & 15u));
    r.next = un;
    return r;
}

// Decoder state of the paper, (p, n, c, z), with c refined to the data unit inside the MCU
// (two decoders inside different luminance units of a 4:2:0 MCU agree on the component but
// not on what follows) and n kept as completed data units (see SInfo).
struct Lane {
    uint32_t p;    // bit position in the unstuffed stream of the next syntax element (kept by the window inside the
                   // decode loops, written back when they end)
    uint32_t u;    // data unit inside the MCU
    uint32_t z;    // zig-zag index of the next coefficient (0 = a DC symbol is next)
    uint32_t nb;   // data units completed since the counter was last cleared
    // pipeline registers (prime)
    uint32_t e;    // table entry already read for the symbol at p (possibly a first-level escape)
    uint32_t base; // table that entry came from
    // synchronisation pass with two symbols per step (decode_span_sync_pairs)
    uint32_t pb;   // pair byte read for the symbol at p, as if that symbol came from unit u's AC table
};

// Window on the stream: two consecutive big-endian words and the offset of the next unread bit in the
// first; `peek` is the 32 bits that start there (a codeword has at most 16 bits, its value at most 16).
struct BitWin {
    uint32_t hi, lo;
    uint32_t o;      // 0..31
    uint32_t peek;
    uint32_t next;   // cursor of the word held in `ahead`, in the units of the Fetch functor; hi is word next - 2
    uint32_t ahead;  // the word after `lo`, fetched one refill early so that its latency is hidden
    uint32_t origin; // bit position in the stream of the word with cursor 0
};

// bit position of the next unread bit
JPGD_HD uint32_t win_pos(const BitWin& w) { return w.origin + ((w.next - 2u) << 5) + w.o; }
// the window has reached bit `limit` (a multiple of 32) as soon as its cursor `next` has reached this value
JPGD_HD uint32_t win_stop(const BitWin& w, uint32_t limit) { return ((limit - w.origin) >> 5) + 2u; }

// per-image constants of the scan syntax
struct Syntax {
    const UnitRow* rows;  // one per data unit of the MCU
    uint32_t upm;         // units per MCU
    const uint32_t* pair_of_unit = nullptr;  // per data unit: offset of its AC table's pair bytes (kernels that use them)
};

JPGD_HD uint32_t win_peek(const BitWin& w) {
    return (uint32_t)(((((uint64_t)w.hi << 32) | (uint64_t)w.lo) << w.o) >> 32);
}

// `cursor` addresses the 32-bit word that holds bit p
template <class Fetch>
JPGD_HD void win_init(BitWin& w, uint32_t p, uint32_t cursor, Fetch fetch) {
    w.hi = fetch(cursor);
    w.lo = fetch(cursor + 1u);
    w.o = p & 31u;
    w.peek = win_peek(w);
    w.next = cursor + 2u;
    w.ahead = fetch(w.next);
    w.origin = (p & ~31u) - (cursor << 5);
}

// Starts the pipeline: after (p, u, z) and the window are set, read the entry of the symbol at p.
template <class LutPtr>
JPGD_HD void prime(Lane& l, const BitWin& w, const Syntax& sx, LutPtr lut) {
    const uint32_t tb_dc = sx.rows[l.u == 0u ? sx.upm - 1u : l.u - 1u].tb_dc_next;
    l.base = l.z == 0u ? tb_dc : sx.rows[l.u].tb_ac;
    l.e = lut[l.base + (w.peek >> (32 - kLutK))];
}

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

// One step of the pipeline, shared by both passes.  Unpacks the entry in hand, moves the window and
// (z, u) past the symbol, and requests the entry of the next symbol (or, for an escape, the second-level
// entry of the same symbol).  What the passes do with the symbol itself comes after, in the shadow of
// that request.
struct Step {
    uint32_t peek;   // window as the symbol saw it
    uint32_t total, size, adv;  // bits taken, value bits among them, zig-zag slots covered
    bool esc;        // first-level escape: nothing was consumed, the state did not change
    bool is_dc;
    bool done;       // the symbol completed its data unit
    bool need;       // the window moved on by a word
    uint32_t z;      // zig-zag index the symbol started at
    uint32_t dcmul;  // of the data unit the symbol belongs to
};

// The row of the current unit is read at the top of the step and used at its end (which table the next entry comes
// from); the next stream word is asked for in the middle and used in the next step; the table entry is asked for
// last and is what the next step starts with.  Nothing but the entry and the window is carried from step to step
// in registers.
template <class Fetch, class LutPtr>
JPGD_HD Step step_and_request(Lane& l, BitWin& w, const Syntax& sx, Fetch fetch, LutPtr lut) {
    Step s;
    const UnitRow old = sx.rows[l.u];
    const uint32_t e = l.e;
    s.peek = w.peek;
    s.esc = lut_esc(e);
    const uint32_t ee = s.esc ? 0u : e;
    s.total = lut_total(ee);  // at most 31
    s.size = lut_size(ee);
    s.adv = lut_adv(ee);
    s.is_dc = l.z == 0u;
    s.z = l.z;
    const uint32_t o2 = w.o + s.total;
    s.need = o2 >= 32u;
    // (bits that start no codeword of a DC table take the DC symbol's slot: sync_entry)
    const uint32_t zn = l.z + (s.is_dc && !s.esc && s.adv == 0u ? 1u : s.adv);
    s.done = zn >= 64u;
    // off the chain, without branches: when no word is taken the word already held is read again, when the
    // unit does not change its row is
    w.next += s.need ? 1u : 0u;
    const uint32_t ahead = fetch(w.next);
    l.u = s.done ? old.next : l.u;
    s.dcmul = old.dcmul;
    l.nb += s.done ? 1u : 0u;
    // window past the symbol
    w.o = o2 & 31u;
    w.hi = s.need ? w.lo : w.hi;
    w.lo = s.need ? w.ahead : w.lo;
    w.ahead = ahead;
    w.peek = win_peek(w);
    l.z = s.done ? 0u : zn;
    // request: next symbol from the DC table of the next unit or the AC table of this one; an escape asks
    // the second level of the table it came from
    uint32_t base2 = s.done ? old.tb_dc_next : old.tb_ac;
#if defined(__HIP_DEVICE_COMPILE__)
    // (Only the arm for ordinary entries below uses base2, and the compiler would move the read of the row into that
    // arm and wait for it there; this keeps the read at the top of the step.)
    asm volatile("" : "+v"(base2));
#endif
    const uint32_t nb2 = lut_esc_bits(e);
    const uint32_t sub = (uint32_t)kLutL1 + lut_esc_offset(e) + ((s.peek >> (32 - kLutK - nb2)) & ((1u << nb2) - 1u));
    const uint32_t idx = s.esc ? l.base + sub : base2 + (w.peek >> (32 - kLutK));
    l.base = s.esc ? l.base : base2;
    l.e = lut[idx];
    return s;
}

// One symbol of the synchronisation pass (write = false in Algorithm 2): state, count of completed units
// (inside step_and_request) and the per-component sums of DC differences.
template <class Fetch, class LutPtr>
JPGD_HD void sync_symbol(Lane& l, BitWin& w, int64_t& dcacc, const Syntax& sx, Fetch fetch, LutPtr lut) {
    const Step s = step_and_request(l, w, sx, fetch, lut);
    const int32_t v = symbol_value(s.peek, s.total, s.size);
    const int32_t mul = s.is_dc ? (int32_t)s.dcmul : 0;
    dcacc += (int64_t)v * (int64_t)mul;
}

// Synchronisation pass: decode while the next symbol starts before `limit`.  The lane must have been primed.
template <class Fetch, class LutPtr>
JPGD_HD void decode_span_sync(Lane& l, BitWin& w, uint32_t limit, int64_t& dcacc, const Syntax& sx, Fetch fetch,
                              LutPtr lut) {
    const uint32_t stop = win_stop(w, limit);
    while (w.next < stop) sync_symbol(l, w, dcacc, sx, fetch, lut);
    l.p = win_pos(w);
}

// ---- two symbols per step ---------------------------------------------------------------------------------
// (The kernels' lanes take two symbols per step from tables of their own, sync_span below.  decode_span_sync,
// decode_span_sync_pairs and decode_span_sync_rst say the same on the tables of jpgd_lut.h; the host walk-through runs
// them, and sync_span is held to them.)
// The synchronisation pass needs the state, the unit count and the DC sums, not the coefficients.  So where the
// first-level index of an AC symbol also holds the whole codeword of the AC symbol after it, one step may take
// both: the pair byte of that index (build_pairs) says how many bits the second symbol takes and how many slots it
// covers.  The second symbol is taken only if the first one is an AC symbol that leaves its data unit open (the
// second then belongs to the same unit and the same table); the step is exactly two steps of sync_symbol.
template <class Fetch, class LutPtr, class PairPtr>
JPGD_HD void sync_symbol_pair(Lane& l, BitWin& w, int64_t& dcacc, const Syntax& sx, Fetch fetch, LutPtr lut,
                              PairPtr pairs) {
    const UnitRow row = sx.rows[l.u];
    const uint32_t pair = sx.pair_of_unit[l.u];
    const uint32_t e = l.e;
    const uint32_t peek = w.peek;
    const bool esc = lut_esc(e);
    const uint32_t ee = esc ? 0u : e;
    const uint32_t t1 = lut_total(ee), size = lut_size(ee), a1 = lut_adv(ee);
    const bool is_dc = l.z == 0u;
    const uint32_t zn1 = l.z + (is_dc && !esc && a1 == 0u ? 1u : a1);
    const uint32_t pb = (is_dc || zn1 >= 64u) ? 0u : l.pb;  // (an escape's index has pair byte 0)
    const uint32_t a2c = pb >> 4;
    const uint32_t total = t1 + (pb & 15u);
    const uint32_t zn = zn1 + a2c;
    const bool done = zn >= 64u || a2c == 15u;  // 15: the second symbol is end-of-block
    const uint32_t o2 = w.o + total;  // at most 31 + 20 + 15
    const bool need = o2 >= 32u;
    w.next += need ? 1u : 0u;
    const uint32_t ahead = fetch(w.next);
    l.nb += done ? 1u : 0u;
    w.o = o2 & 31u;
    w.hi = need ? w.lo : w.hi;
    w.lo = need ? w.ahead : w.lo;
    w.ahead = ahead;
    w.peek = win_peek(w);
    l.z = done ? 0u : zn;
    l.u = done ? row.next : l.u;
    uint32_t base2 = done ? row.tb_dc_next : row.tb_ac;
#if defined(__HIP_DEVICE_COMPILE__)
    // (Only the arm for ordinary entries below uses base2, and the compiler would move the read of the row into that
    // arm and wait for it there; this keeps the read at the top of the step.)
    asm volatile("" : "+v"(base2));
#endif
    const uint32_t nb2 = lut_esc_bits(e);
    const uint32_t sub = (uint32_t)kLutL1 + lut_esc_offset(e) + ((peek >> (32 - kLutK - nb2)) & ((1u << nb2) - 1u));
    const uint32_t i1 = w.peek >> (32 - kLutK);
    const uint32_t idx = esc ? l.base + sub : base2 + i1;
    l.base = esc ? l.base : base2;
    l.e = lut[idx];
    // asked as if the next symbol came from the AC table of the unit just left: if the unit is complete the next
    // symbol is a DC symbol and the byte is not looked at
    l.pb = pairs[pair + i1];
    const int32_t v = symbol_value(peek, t1, size);
    dcacc += (int64_t)v * (int64_t)(is_dc ? (int32_t)row.dcmul : 0);
}

// The synchronisation pass with pairs.  A second symbol must start before `limit` like any other: pairs are taken
// while the step starts at least 32 bits before it (a first symbol with a pair byte has at most 20 bits), single
// symbols from there on.  The lane must have been primed; sx.pair_of_unit must be set.
template <class Fetch, class LutPtr, class PairPtr>
JPGD_HD void decode_span_sync_pairs(Lane& l, BitWin& w, uint32_t limit, int64_t& dcacc, const Syntax& sx, Fetch fetch,
                                    LutPtr lut, PairPtr pairs) {
    const uint32_t stop = win_stop(w, limit);
    l.pb = pairs[sx.pair_of_unit[l.u] + (w.peek >> (32 - kLutK))];
#if defined(__HIP_DEVICE_COMPILE__)
    // (Keeps the compiler from merging this read with the one at the end of a step into a single read at the top of
    // the loop, where every step would wait for it: the byte is asked for one step ahead, like the table entry.)
    asm volatile("" : "+v"(l.pb));
#endif
    while (w.next + 1u < stop) sync_symbol_pair(l, w, dcacc, sx, fetch, lut, pairs);
    while (w.next < stop) sync_symbol(l, w, dcacc, sx, fetch, lut);
    l.p = win_pos(w);
}

// ---- the lanes of the synchronisation pass -----------------------------------------------------------------
// The same walk as decode_span_sync, on tables laid out for it in LDS (SyncTables): a 32-bit entry per first-level index
// says at once what its symbol takes, what the symbol behind it takes where the index holds that one's whole codeword
// too (build_pairs), and how many value bits a DC symbol has.  Position and zig-zag index are one register that an entry
// is added to.
//
// What bounds it: a lane's next look-up waits for the one before (about 130 cycles of LDS), and behind that for the
// instructions between an entry's arrival and the next request, 4 cycles each; with several wavefronts on a SIMD, for
// all instructions of a step.  So the words on the way from entry to request are kept few, everything else stands behind
// the request, and an escape (a codeword longer than the index) is followed up without a branch, which would cost a
// lone wavefront more than the instructions it skips: 46 vector instructions and three LDS reads a step where
// sync_symbol_pair takes 62 and five, two thirds of them in front of the request.
// Measured, decode_span_sync_pairs / this (kernels, us): 15360x8640 first kernel 697 / 611, second 890 / 848; 256 images of
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

// Every entry of a DC table covers the one slot of a DC symbol, also where no codeword starts (which takes a bit): the symbol
// behind it comes from the AC table, and with index 0 the lane's state (position, unit, index) would say otherwise to whoever
// takes the chain over.  Such bits are met off the true chain, or in a damaged stream.
constexpr uint32_t kSyncDcSlot = 1u << 9;
// second-level entry (or first-level one that is no escape) of build_lut, with pair byte pb (0: none)
JPGD_HD uint32_t sync_entry(uint32_t e, bool is_dc, uint32_t pb) {
    const uint32_t slots = pb >> 4;
    return (e & kSyncStep) | (is_dc ? kSyncDcSlot : 0u) | (is_dc ? lut_size(e) << 20 : ((pb & 15u) | ((slots == 15u ? kAdvEob : slots) << 9)) << 16);
}
constexpr uint32_t kWriteInside = 1u << 16, kWriteNoCode = 1u << 17;
constexpr int32_t kWriteValue = 1 << 30, kWriteDc = 3 << 29;
JPGD_HD uint32_t write_entry(uint32_t e, bool is_dc) {
    const uint32_t slots = lut_adv(e), size = lut_size(e);
    return (e & kSyncStep) | (is_dc ? kSyncDcSlot : 0u) | (size << 20) | (slots == 0u ? kWriteNoCode : !is_dc && slots != kAdvEob ? kWriteInside : 0u) |
           (uint32_t)(slots == 0u ? 0 : is_dc ? kWriteDc : size != 0u ? kWriteValue : 0);
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
JPGD_HD uint32_t sync_dc_direct(uint32_t a) { return pass_entry<WRITE>(lut_esc(a) ? 1u : a, true, 0u); }

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

// One symbol of the write pass (write = true in Algorithm 2): every non-zero coefficient goes to
// 64*unit + zig-zag index, DC values un-differenced.  `unit` is the index of the data unit being decoded,
// pred0..2 the DC predictors; `flags` collects kSt* bits.  Without branches except around the store itself:
// a wavefront holds lanes in every kind of symbol at once, so each arm of a branch would be walked anyway.
template <class Fetch, class LutPtr, class Store>
JPGD_HD void write_symbol(Lane& l, BitWin& w, uint32_t& unit, int32_t& pred0, int32_t& pred1, int32_t& pred2,
                          const Syntax& sx, Fetch fetch, LutPtr lut, Store store, uint32_t& flags) {
    const Step s = step_and_request(l, w, sx, fetch, lut);
    const bool comp0 = s.dcmul == 1u, comp1 = s.dcmul == (1u << 15);
    // An escape comes out as value 0, size 0, no slot; bits that start no codeword as value 0, size 0, one bit, no
    // slot: neither changes a predictor or passes the test of the store below.
    const int32_t value = symbol_value(s.peek, s.total, s.size);
    const bool dc = s.is_dc;
    const int32_t pred = (comp0 ? pred0 : (comp1 ? pred1 : pred2)) + value;
    pred0 = dc && comp0 ? pred : pred0;
    pred1 = dc && comp1 ? pred : pred1;
    pred2 = dc && !comp0 && !comp1 ? pred : pred2;
    // where the symbol ends: a coefficient sits in the last slot it covers (after its run of zeros); a DC symbol ends
    // in slot 0, or, if it covers none, before it
    const uint32_t zn = s.z + s.adv;
    const uint32_t at = zn - 1u;
    if ((dc || s.size != 0u) && at < 64u) store(unit, at, (int16_t)(dc ? pred : value));  // (a DC symbol of size 0 still yields the predictor)
    // no codeword starts with these bits; or a coefficient or a run of sixteen zeros (not end-of-block,
    // which may be coded anywhere) that runs past the end of the unit
    const bool bad = (s.adv == 0u && !s.esc) || (zn > 64u && s.adv != kAdvEob);
    flags |= bad ? kStInvalid : 0u;
    unit += s.done ? 1u : 0u;
}

// Write pass: the same walk as the synchronisation pass, up to the image's last data unit.
template <class Fetch, class LutPtr, class Store>
JPGD_HD void decode_span_write(Lane& l, BitWin& w, uint32_t limit, uint32_t& unit, uint32_t total_units,
                               int32_t& pred0, int32_t& pred1, int32_t& pred2, const Syntax& sx, Fetch fetch,
                               LutPtr lut, Store store, uint32_t& flags) {
    const uint32_t stop = win_stop(w, limit);
    while (w.next < stop && unit < total_units) write_symbol(l, w, unit, pred0, pred1, pred2, sx, fetch, lut, store, flags);
    l.p = win_pos(w);
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

// the window moves to bit B (a multiple of 8) and the decoder starts a fresh MCU there
template <class Fetch, class LutPtr>
JPGD_HD void move_to_interval(Lane& l, BitWin& w, uint32_t B, const Syntax& sx, Fetch fetch, LutPtr lut) {
    l.z = 0u;
    l.u = 0u;
    win_init(w, B, (B - w.origin) >> 5, fetch);
    prime(l, w, sx, lut);
}

// after a symbol: has the decoder reached the padding in front of the interval that starts at B, or passed B?
JPGD_HD bool at_interval_end(const BitWin& w, uint32_t pos, uint32_t B) {
    if (pos >= B) return true;
    const uint32_t r = B - pos;
    return r <= 7u && (~w.peek >> (32u - r)) == 0u;
}

// Where the fast part of a span ends when the next interval starts at B: a symbol that starts before `calm` ends more
// than 7 bits before B (it has at most 31 bits), so nothing has to be checked on the way there.  As a window cursor.
JPGD_HD uint32_t calm_stop(const BitWin& w, uint32_t B, uint32_t limit) {
    uint32_t calm = limit;
    if (B != kNoBoundary) {
        const uint32_t c = B >= 40u ? (B - 39u) & ~31u : 0u;
        calm = c < limit ? c : limit;
    }
    return calm > w.origin ? win_stop(w, calm) : 0u;
}

// Synchronisation pass over a stream with restart intervals.  `crossed` is set when a symbol of this span
// started an interval (dcacc then holds the sums since the last such symbol).
// A fast loop up to the neighbourhood of the next interval start, then a careful loop.  (The single loop of the
// write pass below was measured here too: the overflow rounds are a chain of dependent symbols in a lone
// wavefront, and the extra tests per symbol cost them more -- 4096x4096 with one interval per MCU row: 0.93
// against 0.78 ms -- than walking a span twice costs the few wavefronts that meet an interval start.)
template <class Fetch, class LutPtr, class BWord>
JPGD_HD void decode_span_sync_rst(Lane& l, BitWin& w, uint32_t limit, int64_t& dcacc, uint32_t& crossed, const Syntax& sx,
                                  Fetch fetch, LutPtr lut, BWord bword) {
    uint32_t from = win_pos(w);
    for (;;) {
        const uint32_t B = next_boundary(from, limit + 64u, bword);
        const uint32_t stop = calm_stop(w, B, limit);
        while (w.next < stop) sync_symbol(l, w, dcacc, sx, fetch, lut);
        if (B == kNoBoundary) break;
        uint32_t pos = win_pos(w);
        bool next_interval = false;
        while (pos < limit) {
            if (pos == B) {  // this symbol starts the interval
                dcacc = 0;
                crossed = 1u;
                from = B + 1u;
                next_interval = true;
                break;
            }
            sync_symbol(l, w, dcacc, sx, fetch, lut);
            pos = win_pos(w);
            if (at_interval_end(w, pos, B)) {
                move_to_interval(l, w, B, sx, fetch, lut);
                pos = B;
            }
        }
        if (!next_interval) break;
    }
    l.p = win_pos(w);
}

// The same over a stream with restart intervals (rules: decode_span_sync_rst below, which this follows step by step).
// Boundaries are positions in the image's stream: a position there plus `org` is a bit of `word`.  start(p): sync_start at
// bit p with u = z = 0; span(limit): sync_span.
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

// The write pass's lanes over a stream with restart intervals (rules: decode_span_write_rst below).  `org` as in
// sync_span_rst; *flags: kStInvalid where an interval starts at another unit than it should.
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

// Write pass over a stream with restart intervals: the predictors return to zero where an interval starts.
// An interval holds units_per_interval data units (all but the last of the scan): a start reached at any
// other unit count means damaged data and is flagged.
// One loop for all lanes: a lane near an interval start does its checks before and after the same write_symbol the
// others execute.  With a fast loop and a careful loop one after the other, a wavefront in which a few lanes meet
// an interval start walks its span up to three times (the fast loop for the others, the careful one, the fast
// one again for what follows the start); the write kernel, whose wavefronts all have full spans to decode, is a
// third faster this way on streams with one interval per MCU row.
template <class Fetch, class LutPtr, class Store, class BWord>
JPGD_HD void decode_span_write_rst(Lane& l, BitWin& w, uint32_t limit, uint32_t& unit, uint32_t total_units,
                                   uint32_t units_per_interval, int32_t& pred0, int32_t& pred1, int32_t& pred2,
                                   const Syntax& sx, Fetch fetch, LutPtr lut, Store store, uint32_t& flags, BWord bword) {
    uint32_t B = next_boundary(win_pos(w), limit + 64u, bword);
    uint32_t stop = calm_stop(w, B, limit);
    while (unit < total_units) {
        const bool near = w.next >= stop;
        if (near) {
            if (B == kNoBoundary) break;
            const uint32_t pos = win_pos(w);
            if (pos >= limit) break;
            if (pos == B) {
                pred0 = pred1 = pred2 = 0;
                if (unit % units_per_interval != 0u) flags |= kStInvalid;
                B = next_boundary(B + 1u, limit + 64u, bword);
                stop = calm_stop(w, B, limit);
                continue;
            }
        }
        write_symbol(l, w, unit, pred0, pred1, pred2, sx, fetch, lut, store, flags);
        if (near && at_interval_end(w, win_pos(w), B)) move_to_interval(l, w, B, sx, fetch, lut);
    }
    l.p = win_pos(w);
}

}  // namespace jpgd
