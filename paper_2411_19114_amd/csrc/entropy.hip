// GPU Huffman entropy decoder for baseline JPEG (T.81 F.2.2), gfx950.
//
// The first half of the "Decode" functional unit (PREBA section 4.2, Table 1).
// The FPGA decodes one stream serially per compute unit; here one workgroup owns
// a run of whole restart intervals (T.81 E.2.4) of one image, or a window of a stream
// that has none:
//
//   1. scan_restart_markers counts the RSTn markers in fixed windows of every
//      image's entropy-coded segment, so that a workgroup starting at the first
//      marker of its window knows which restart interval (hence which MCU) it
//      starts at, without any serial pass over the stream.
//   2. decode_entropy stages a chunk of the stream in LDS with byte stuffing
//      (FF 00) and markers removed and the interval starts marked, then decodes
//      it in one of two ways:
//      - short intervals: one lane per restart interval, a single sequential pass
//        that writes coefficients directly (start state and MCU index are known);
//      - long intervals or none: every lane takes a fixed-size subsequence and
//        decodes from a guessed state (code-word boundary, block 0 of an MCU, DC
//        coefficient); lane j then re-decodes from the end state lane j-1 reached
//        until no end state changes.  Lane 0 starts from a known state, so the
//        fixed point is the sequential decode, exactly.  A prefix sum of completed
//        blocks gives every lane its block index, a last pass writes coefficients,
//        and a segmented scan turns DC differences into absolute values.
//      - calls with little data (small windows, kHyp): the states at the subsequence
//        borders inside restart intervals are found by phase hypotheses in two passes
//        (the by_hypotheses branch) instead of by iteration, then written as above.
//   3. Streams without restart markers are mostly cut into windows that several workgroups decode
//      side by side (resolve_streams and the kernels after it, which run on either side of
//      decode_entropy).  decode_entropy iterates over those that are not (StreamCut in api.cpp) or
//      whose windows cannot be joined.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/prep.h"
#include "kernels.h"
#include "prep_internal.h"

namespace prep {

namespace {

constexpr int kT = kDecodeThreads;
constexpr int kPadShift = 4;                        // rows of 16 words (= one subsequence) + 1 (copy of the next)
constexpr int kCleanWords = kChunkRaw / 4 + kT + 16;  // destuffed stream, the rows' last words, zero tail
constexpr int kMaskWords = kChunkRaw / 32 + 2;      // one bit per clean byte
constexpr int kMaxBoundaries = 1024;                // listed interval starts per chunk
constexpr uint32_t kShortInterval = kLongIntervalBytes;  // mean clean bytes up to which a lane takes a whole interval
constexpr uint32_t kNoMarker = 0xFFFFFFFFu;
constexpr uint32_t kSubBits = kSubseqBytes * 8;
static_assert(kSubseqBytes == 64 && (kSubseqBytes / 4) == (1 << kPadShift), "one 64-bit keep mask per lane");
static_assert(kT == 256, "a row's number fits a byte; four waves");

// Lookup entry of a Huffman code (16 bits):
//   bits 4..0   code length + number of appended bits (1..31); 0 = search the code lists
//   bits 8..5   number of appended bits
//   bits 15..9  zig-zag advance - 1 (DC 0, AC run, ZRL 15, EOB 127).  Added to the zig-zag index it
//               gives the index k of the symbol's coefficient, which must not exceed 63 except
//               for EOB, whose coefficient is the block's last: k <= 63 is in order, 64 <= k < 128
//               is a run past the block's end, k >= 128 is EOB (bit 6 of k tells)
// (the first field shifted to the top of a word leaves nothing of the others: see BitCursor)
constexpr uint32_t kEobAdvance = 127;
// bits that are no code word: 16 bits, ends the block, and is refused like a run past its end
constexpr uint32_t kInvalidEntry = 16u | (64u << 9);
constexpr uint32_t kSearchEntry = 0;
// the same in a DC table, where it must not move the index: as many appended bits as no DC code has
constexpr uint32_t kInvalidDcEntry = 16u | (15u << 5);
constexpr uint32_t entry_bits(uint32_t e) { return e & 31u; }
constexpr uint32_t entry_appended(uint32_t e) { return (e >> 5) & 15u; }
constexpr uint32_t entry_advance(uint32_t e) { return e >> 9; }

// One lookup resolves codes of every length.  Canonical codes grow longer with their value
// (T.81 Annex C), so the codes of more than ten bits lie at the top of the code space: below
// kFinePrefixes ten-bit prefixes there is an entry for each prefix, above an entry for each
// sixteen-bit word.  With a = the next sixteen bits the entry is number max(a / 64, a - 63 *
// kFinePrefixes): the two meet where the fine part begins, and either side of it the other
// is the smaller.  Eight fine prefixes: the codes of T.81 Annex K need five of each AC table, codes
// made for photographs and noise of qualities 50 to 95 at most four.  A prefix below that still
// begins a longer code (codes far from any image's statistics) has kSearchEntry.
// With a second level for the codes of more than ten bits, read in a branch of its own, 1.6 % of
// the symbols took that branch but half of all iterations of a wave of 64 lanes did.
constexpr uint32_t kFinePrefixes = 1016;
constexpr uint32_t kLookupEntries = kFinePrefixes + 64u * (1024u - kFinePrefixes);

// What a writing pass needs of an image's four tables
struct alignas(16) HuffCodes {
    // the tables (DC luma, AC luma, DC chroma, AC chroma) interleaved: entry (number << 2) | table
    uint16_t one[4 * kLookupEntries];
    int32_t first[4][17];            // first code of each length
    int32_t count[4][17];            // BITS
    int32_t valptr[4][17];           // index of the first symbol of each length
    uint8_t huffval[4][256];
};
// and what the passes that only find states do: entries for as many whole symbols as the ten bits
// of a prefix hold the codes of (their bits, and their advances together; no values), so that a
// lookup goes on by 1.6 to 1.9 symbols.  A DC symbol is followed by those of its component's AC
// table.  The symbols stop
//   - behind an EOB (the advance is kEobAdvance then),
//   - where the symbols before the last advance by more than kRunLead together: up to
//     zig-zag index 62 - kRunLead none of them ends the block,
//   - with what does not fit the entry's fields.
// All but the last end within the ten bits.  Prefixes of longer codes have their single symbol.
struct alignas(16) HuffTables : HuffCodes {
    uint16_t run[4 * kLookupEntries];
};
constexpr int32_t kRunLead = 16;
constexpr uint32_t kRunLeadBits = 9;  // most bits of the symbols before the last

// Rows (subsequences) that a round of the iteration decodes, and every row's blocks
struct RowLists {
    uint32_t from[kT];
    uint16_t blocks[kT];
    uint8_t row[kT];
};

// kHyp, kRuns: see decode_entropy
template <bool kHyp, bool kRuns>
struct DecodeShared {
    // The destuffed stream, big-endian packed (bit 31 of a word is the earliest bit).  In the
    // subsequence passes every 16 words (a subsequence) are followed by a copy of the next
    // word: rows of 17, so that lanes that read at similar offsets of their subsequences hit
    // different LDS banks, and a lane's reads stay in its row (see clean_row_of_bit).
    uint32_t clean[kCleanWords];
    uint32_t bmask[kMaskWords];      // bit q set: a restart interval begins at clean byte q
    uint32_t next_boundary[kT + 1];  // first interval start at or after the lane's subsequence
    // Interval starts of the chunk in order (clean byte offsets), for the pass that takes an
    // interval a lane; the others need to know which of a lane's 64 raw bytes survived destuffing
    // (and the hypothesis passes use the list's place for states: there a lane keeps it in registers)
    union {
        uint16_t bpos[kMaxBoundaries];
        unsigned long long keep[kHyp ? 1 : kT];
        RowLists rows_here;
    };
    std::conditional_t<kHyp, uint8_t, RowLists> rows_there;
    __device__ RowLists &rows()
    {
        if constexpr (kHyp) return rows_here;
        else return rows_there;
    }
    std::conditional_t<kRuns, HuffTables, HuffCodes> tab;
    uint32_t keep_off[kT + 1];       // clean offset of the lane's first surviving byte
    uint32_t state[kT];              // end state of every subsequence
    uint32_t scan_a[kT / 64 + 1];    // per-wave totals for workgroup scans
    int32_t dc_val[kT / 64 + 1];
    int32_t dc_flag[kT / 64 + 1];
    uint32_t bcast[8];
};

// Workgroups that a compute unit's 160 KB of LDS hold: they get theirs in units of 1280 bytes
constexpr uint32_t workgroups_by_lds(size_t bytes) { return (160u << 10) / 1280u / (uint32_t)((bytes + 1279u) / 1280u); }

__device__ inline uint32_t pack_state(uint32_t p, uint32_t blk, uint32_t zz)
{
    return (p << 9) | (blk << 6) | zz;
}

// ---- workgroup-wide helpers (kT threads, wave64) ---------------------------

__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

// exclusive prefix sum over the workgroup; *total receives the sum
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t *wave_tot, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    __syncthreads();
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kT / 64; w++) {
        uint32_t t = wave_tot[w];
        if (w < wave) base += t;
        tot += t;
    }
    *total = tot;
    return base + inc - v;
}

// sum over the workgroup
__device__ inline uint32_t block_sum(uint32_t v, uint32_t *wave_tot)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wave_tot[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < kT / 64; w++) tot += wave_tot[w];
    return tot;
}

// Segmented running sum (value, reset flag): a reset discards what came before.
// Returns the value carried INTO this lane (exclusive); carry_in seeds lane 0.
__device__ inline int32_t block_seg_excl_scan(int32_t v, int32_t f, int32_t carry_in,
                                              int32_t *wave_val, int32_t *wave_flag,
                                              int32_t *carry_out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t iv = v, ifl = f;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int32_t ov = __shfl_up(iv, d, 64);
        int32_t of = __shfl_up(ifl, d, 64);
        if (lane >= d) {
            if (!ifl) iv += ov;
            ifl |= of;
        }
    }
    __syncthreads();
    if (lane == 63) { wave_val[wave] = iv; wave_flag[wave] = ifl; }
    __syncthreads();
    int32_t cv = carry_in, all_v = carry_in;
#pragma unroll
    for (int w = 0; w < kT / 64; w++) {
        int32_t wv = wave_val[w], wf = wave_flag[w];
        int32_t nv = wf ? wv : all_v + wv;
        if (w < wave) cv = nv;
        all_v = nv;
    }
    *carry_out = all_v;
    int32_t pv = __shfl_up(iv, 1, 64);
    int32_t pf = __shfl_up(ifl, 1, 64);
    if (lane == 0) return cv;
    return pf ? pv : cv + pv;
}

// ---- Huffman tables (T.81 Annex C) --------------------------------------------

// canonical search among the code lengths lo..hi for the code that starts `peek16`
__device__ inline bool canonical_lookup(const HuffCodes &T, int t, uint32_t peek16, int lo, int hi,
                                        uint32_t *len, uint32_t *sym)
{
#pragma unroll 1
    for (int l = lo; l <= hi; l++) {
        const int32_t c = (int32_t)(peek16 >> (16 - l)) - T.first[t][l];
        if (c >= 0 && c < T.count[t][l]) {
            *len = (uint32_t)l;
            *sym = T.huffval[t][(T.valptr[t][l] + c) & 255];
            return true;
        }
    }
    return false;
}

__device__ inline uint32_t make_entry(bool ac, uint32_t sym, uint32_t len)
{
    uint32_t s = sym & 15u, advance;
    if (!ac) {
        if (sym > 11u) return kSearchEntry;  // no such DC category in baseline
        advance = 0;
    } else if (s == 0) {
        advance = (sym >> 4) == 15u ? 15u : kEobAdvance;  // ZRL, otherwise end of block
    } else {
        advance = sym >> 4;
    }
    return (advance << 9) | (s << 5) | (len + s);
}

// the run entries, or the single ones where no others are kept
__device__ __forceinline__ const uint16_t *run_entries(const HuffTables &T) { return T.run; }
__device__ __forceinline__ const uint16_t *run_entries(const HuffCodes &T) { return T.one; }

// number of the lookup entry for the next bits `win` of the stream
__device__ __forceinline__ uint32_t lookup_number(uint32_t win)
{
    return (uint32_t)max((int32_t)(win >> 22), (int32_t)(win >> 16) - (int32_t)(63u * kFinePrefixes));
}

// Expands the four tables (all lanes of the workgroup must call).
__device__ inline void build_tables(HuffCodes &T, const uint8_t *file, const ImageRec &R)
{
    const int tid = threadIdx.x;
    if (tid < 4) {
        const uint8_t *b = file + R.dht_off[tid];
        int32_t bits[16];
#pragma unroll
        for (int l = 0; l < 16; l++) bits[l] = b[l];
        int32_t code = 0, k = 0;
        T.first[tid][0] = T.count[tid][0] = T.valptr[tid][0] = 0;
#pragma unroll
        for (int l = 1; l <= 16; l++) {
            const int32_t c = bits[l - 1];
            T.first[tid][l] = code;
            T.count[tid][l] = c;
            T.valptr[tid][l] = k;
            code = (code + c) << 1;
            k += c;
        }
    }
    for (int t = 0; t < 4; t++) {
        const uint32_t nval = min(R.dht_nval[t], 256u);
        for (uint32_t i = tid; i < 256u; i += kT) T.huffval[t][i] = i < nval ? file[R.dht_off[t] + 16 + i] : 0;
    }
    __syncthreads();
    for (int t = 0; t < 4; t++) {
        // the sixteen-bit words below end[l - 1] begin with a code of at most l bits
        uint32_t end[16];
#pragma unroll
        for (int l = 1; l <= 16; l++) end[l - 1] = (uint32_t)(T.first[t][l] + T.count[t][l]) << (16 - l);
        for (uint32_t i = tid; i < kLookupEntries; i += kT) {
            const bool fine = i >= kFinePrefixes;
            const uint32_t a = fine ? i + 63u * kFinePrefixes : i << 6;
            uint32_t l = 1;
#pragma unroll
            for (int k = 0; k < 16; k++) l += a >= end[k] ? 1u : 0u;
            uint32_t e = t & 1 ? kInvalidEntry : kSearchEntry;  // past the last code
            if (l <= 16u) {
                const uint32_t c = (a >> (16u - l)) - (uint32_t)T.first[t][l];
                e = fine || l <= 10u ? make_entry(t & 1, T.huffval[t][((uint32_t)T.valptr[t][l] + c) & 255u], l) : kSearchEntry;
            }
            T.one[(i << 2) | (uint32_t)t] = (uint16_t)e;
        }
    }
    __syncthreads();
}

// The run entry of prefix i from its single entry e; one(n) = single entry number n of the table that the
// prefix's further symbols are of.
template <typename One>
__device__ __forceinline__ uint32_t run_entry(uint32_t e, uint32_t i, One one)
{
    if (e == kSearchEntry || e == kInvalidEntry) return e;
    uint32_t bits = entry_bits(e), advance = entry_advance(e);
    // (a symbol has at least one bit: the loop ends)
    while (advance != kEobAdvance && bits <= kRunLeadBits) {
        const int32_t lead = (int32_t)advance + 1;  // how far the zig-zag index has come by the symbols so far
        if (lead > kRunLead) break;
        const uint32_t n = one(lookup_number(i << (22 + bits)));
        // the next code lies within the prefix?  (the zeros behind it are not the stream's)
        if (n == kSearchEntry || n == kInvalidEntry || bits + entry_bits(n) - entry_appended(n) > 10u) break;
        if (bits + entry_bits(n) > 31u) break;
        bits += entry_bits(n);
        advance = entry_advance(n) == kEobAdvance ? kEobAdvance : (uint32_t)lead + entry_advance(n);
    }
    return (advance << 9) | bits;
}

// The run entries of all tables from the single ones of these and, for a DC table, of the AC table
// behind it (all lanes of the workgroup must call).
__device__ inline void build_runs(HuffTables &T)
{
    for (int t = 0; t < 4; t++) {
        for (uint32_t i = threadIdx.x; i < kLookupEntries; i += kT) {
            uint32_t e = T.one[(i << 2) | (uint32_t)t];
            if (i < kFinePrefixes) e = run_entry(e, i, [&](uint32_t n) { return (uint32_t)T.one[(n << 2) | (uint32_t)(t | 1)]; });
            T.run[(i << 2) | (uint32_t)t] = (uint16_t)e;
        }
    }
    __syncthreads();
}

// Part `part` of an image's table t (lookup and run entries, code lists), straight from the DHT bytes
// into a slot of expanded tables, an entry a lane.  A run's further symbols are found among the codes like
// its first, so that no lane waits for the others' entries.  (One workgroup a table, entries looked up in
// those made before, was what small calls waited for in this kernel: 11.5 us, 5.2 now; 33 sets of
// tables 13.8 -> 11.2, 64 16.1 -> 12.0 against whole tables made like this.)  Run entries cost most and are left
// out where no kernel of the call reads them.  All lanes of the workgroup must call.
constexpr uint32_t kTableParts = (kLookupEntries + kT - 1) / kT;
struct CodeLists {
    int32_t first[17], count[17], valptr[17];
    uint32_t end[16];  // the sixteen-bit words below end[l - 1] begin with a code of at most l bits
    uint8_t huffval[256];
};
__device__ inline void expand_table(const uint8_t *file, const ImageRec &R, int t, uint32_t part, bool runs, HuffTables *dst)
{
    __shared__ CodeLists lists[2];  // of table t, and of the AC table behind it
    const int tid = threadIdx.x;
    for (int k = 0; k < 2; k++) {
        const int of = k ? t | 1 : t;
        lists[k].huffval[tid] = (uint32_t)tid < min(R.dht_nval[of], 256u) ? file[R.dht_off[of] + 16 + tid] : 0;
    }
    if (tid < 2) {
        const uint8_t *b = file + R.dht_off[tid ? t | 1 : t];
        CodeLists &L = lists[tid];
        int32_t bits[16];
#pragma unroll
        for (int l = 0; l < 16; l++) bits[l] = b[l];
        int32_t code = 0, k = 0;
        L.first[0] = L.count[0] = L.valptr[0] = 0;
#pragma unroll
        for (int l = 1; l <= 16; l++) {
            const int32_t c = bits[l - 1];
            L.first[l] = code;
            L.count[l] = c;
            L.valptr[l] = k;
            L.end[l - 1] = (uint32_t)(code + c) << (16 - l);
            code = (code + c) << 1;
            k += c;
        }
    }
    __syncthreads();
    // lookup entry number i of table t or t | 1
    auto entry = [&](const CodeLists &L, int ac, uint32_t i) -> uint32_t {
        const bool fine = i >= kFinePrefixes;
        const uint32_t a = fine ? i + 63u * kFinePrefixes : i << 6;
        uint32_t l = 1;
#pragma unroll
        for (int k = 0; k < 16; k++) l += a >= L.end[k] ? 1u : 0u;
        if (l > 16u) return ac ? kInvalidEntry : kSearchEntry;  // past the last code
        const uint32_t c = (a >> (16u - l)) - (uint32_t)L.first[l];
        return fine || l <= 10u ? make_entry(ac != 0, L.huffval[((uint32_t)L.valptr[l] + c) & 255u], l) : kSearchEntry;
    };
    const uint32_t i = part * (uint32_t)kT + (uint32_t)tid;
    if (i < kLookupEntries) {
        const uint32_t e = entry(lists[0], t & 1, i);
        dst->one[(i << 2) | (uint32_t)t] = (uint16_t)e;
        if (runs)
            dst->run[(i << 2) | (uint32_t)t] =
                (uint16_t)(i < kFinePrefixes ? run_entry(e, i, [&](uint32_t n) { return entry(lists[1], 1, n); }) : e);
    }
    if (part != 0) return;
    if (tid < 17) {
        dst->first[t][tid] = lists[0].first[tid];
        dst->count[t][tid] = lists[0].count[tid];
        dst->valptr[t][tid] = lists[0].valptr[tid];
    }
    dst->huffval[t][tid] = lists[0].huffval[tid];
}

// the expanded tables of an image with a table slot, or the part of them that a writing pass
// needs, into LDS (a barrier has to follow)
template <typename Tables>
__device__ inline void load_tables(Tables &tab, const uint4 *__restrict__ tables, uint32_t slot)
{
    constexpr uint32_t units = sizeof(Tables) / 16, all = sizeof(HuffTables) / 16;
    uint4 *dst = reinterpret_cast<uint4 *>(&tab);
#pragma unroll
    for (uint32_t i = threadIdx.x; i < units; i += kT) dst[i] = tables[(size_t)slot * all + i];
}

// ---- bit-level decoding ------------------------------------------------------

struct Geometry {
    uint32_t bpm;        // blocks per MCU
    uint32_t n_luma;     // luma blocks per MCU (blocks >= n_luma use the chroma tables)
    uint32_t ri_blocks;  // blocks per restart interval, 0 = none
    uint32_t n_blocks;   // blocks in the image
    // The symbol loops keep the block's place in the MCU as slot = 5 * block, so that one field
    // extract gives the next block's slot (wrapping at the MCU's end) and another whether a
    // block uses the chroma tables:
    uint32_t next_slot;  // bits [slot, slot + 5): slot of the block after the one at slot
    uint32_t chroma_at;  // bits [slot, slot + 3): 4 if the block at slot uses the chroma tables, else 0
                         // (twice the number of its DC table)
    __device__ void set_slots()
    {
        next_slot = chroma_at = 0;
        for (uint32_t b = 0; b < bpm; b++) {
            next_slot |= (5u * ((b + 1u) % bpm)) << (5u * b);
            chroma_at |= (b >= n_luma ? 4u : 0u) << (5u * b);
        }
    }
};
// (an MCU holds at most six blocks, luma 2 x 2 and two chroma: six 5-bit fields fit a word)

__device__ __forceinline__ uint32_t slot_of_block(uint32_t blk) { return 5u * blk; }
__device__ __forceinline__ uint32_t block_of_slot(uint32_t slot) { return (slot * 13u) >> 6; }  // slot / 5 for slot <= 25

__device__ inline uint32_t comp_of_block(const Geometry &g, uint32_t blk_in_mcu)
{
    return blk_in_mcu < g.n_luma ? 0u : blk_in_mcu - g.n_luma + 1u;
}

// first interval start at or after clean byte q (in bits), limit if none
template <bool kHyp, bool kRuns>
__device__ inline uint32_t boundary_from(const DecodeShared<kHyp, kRuns> &S, uint32_t q, uint32_t limit_bits)
{
    const uint32_t j = q >> 6;
    if (j >= (uint32_t)kT) return limit_bits;
    unsigned long long m = ((unsigned long long)S.bmask[2 * j + 1] << 32) | S.bmask[2 * j];
    m >>= (q & 63);
    uint32_t r = m ? q + (uint32_t)__builtin_ctzll(m) : S.next_boundary[j + 1];
    r = r > 0x0FFFFFFFu ? limit_bits : r * 8u;
    return r < limit_bits ? r : limit_bits;
}

// Per-lane state of a writing pass.  Only scalar members and no indexing by a run-time
// value: the struct must stay in registers (a private-memory copy would make every
// iteration of the decode loop wait for its coefficient stores).
struct WriteCtx {
    int16_t *coef;         // this image's first block
    uint32_t side_rel;     // coef + side_rel = this image's DC differences, one int16 per block
    uint32_t block;        // absolute index of the block being decoded
    int32_t iv_rem;        // blocks left before a restart boundary has to come (0: it comes next)
    int32_t bad;
};

// The rarest part of a lookup: a code that the lookup table refers to the code lists.
__device__ __forceinline__ uint32_t lookup_by_search(const HuffCodes &T, uint32_t tsel, uint32_t win)
{
    uint32_t len, sym, e = kSearchEntry;
    if (canonical_lookup(T, (int)tsel, win >> 16, 11, 16, &len, &sym)) e = make_entry(tsel & 1u, sym, len);
    return e != kSearchEntry ? e : (tsel & 1u) ? kInvalidEntry : kInvalidDcEntry;
}

// Entry for the next bits `win` in a table of `entries`; tb = twice the table's number
__device__ __forceinline__ uint32_t look_up(const uint16_t *entries, uint32_t tb, uint32_t win)
{
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(entries) + (lookup_number(win) << 3) + tb);
}

// Whether a rare branch is worth entering, or a loop for all lanes is: true if x is for any of the
// wave's active lanes
__device__ __forceinline__ bool wave_any(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0; }

// Word w of the destuffed stream lives at index w + (w >> kPadShift) of DecodeShared::clean in
// the subsequence passes: rows of seventeen words, a subsequence's sixteen and a copy of the
// first word of the next.  A lane that decodes subsequence r (from wherever in it to the first
// symbol boundary at or past its end) uses no word beyond that copy, so all its reads are at
// index w + r with r fixed: one add instead of the row arithmetic, and lanes that are equally
// far into their subsequences still read from different banks.  (The words it merely
// prefetches, up to two further, lie in the next row at the wrong place and are never used.)
__device__ __forceinline__ uint32_t clean_row_of_bit(uint32_t p)
{
    static_assert(kSubseqBytes * 8 == 1 << 9 && kPadShift == 4, "bit >> 9 = subsequence = row");
    return p >> 9;
}

// A place in the stream and the next 32 bits there.  The stream words around it are kept in
// registers (an entry's bits are fewer than a word's, so at most one new word is needed a symbol, and it
// is fetched a symbol ahead of its use).  The bit offset is counted down from the next word's
// first bit, in the top five bits of n32, so that the subtraction of a symbol's bits borrows
// exactly where a new word begins, and the offset is the shift that V_ALIGNBIT_B32 takes.
struct BitCursor {
    uint32_t w;              // ceil(position / 32)
    uint32_t n32;            // (32 w - position) << 27
    uint32_t hi, lo, ahead;  // words w - 1, w and w + 1
    uint32_t win;            // the next 32 bits
    __device__ __forceinline__ void start(const uint32_t *words, uint32_t p)
    {
        w = (p + 31u) >> 5;
        n32 = (0u - p) << 27;
        hi = words[p >> 5];  // (word w - 1, or any word where p is a word's first bit)
        lo = words[w];
        ahead = words[w + 1];
        win = __builtin_amdgcn_alignbit(hi, lo, n32 >> 27);
    }
    // past the symbol (or symbols) of entry e
    __device__ __forceinline__ void advance(const uint32_t *words, uint32_t e)
    {
        const bool moved = __builtin_sub_overflow(n32, e << 27, &n32);
        hi = moved ? lo : hi;
        lo = moved ? ahead : lo;
        w += moved ? 1u : 0u;
        win = __builtin_amdgcn_alignbit(hi, lo, n32 >> 27);
        ahead = words[w + 1];
    }
    __device__ __forceinline__ uint32_t position() const { return (w << 5) - (n32 >> 27); }
};

// value of a stored coefficient: appended bits (T.81 F.2.2.4 RECEIVE) and sign extension
// (F.2.2.1 EXTEND); adv = code length + s
__device__ __forceinline__ int32_t coefficient_value(uint32_t win, uint32_t adv, uint32_t s)
{
    // RECEIVE(s) read as a signed field: t < 0 where the first appended bit is 1; 0 for s = 0
    const int32_t t = __builtin_amdgcn_sbfe((int32_t)win, 32u - adv, s);
    // EXTEND: first bit 1: the bits are the value, t + 2^s; first bit 0: 2^s - 1 below them.
    // With m = t >> 31 both are t + ((-2^s) ^ m) + 1.
    return t + (int32_t)((0xFFFFFFFFu << s) ^ (uint32_t)(t >> 31)) + 1;
}

// ---- the symbol loops -----------------------------------------------------------
// One step = one lookup: (writing passes) extract the value and store it, advance position and
// zig-zag index, look the next bits up.  The state carried from one step to the next is the bit
// position, block-in-MCU and zig-zag index only.
//
// The loops are bound by their instructions: a lone wave issues a dependent one every eight cycles
// and an independent one every five, and the waves of a SIMD share its issue.  So the steps are
// written out, in an order in which little waits for the instruction before and a table entry's
// read is under way while the index and the block are settled, and lanes do not leave one by
// one: one loop runs while no lane of the wave is near the end of its span or a restart boundary, one
// that looks at both while none has come there, and all else happens outside, in count_span and
// write_span.  (The compiler's loop for the former, with its masks, copies and branches, took 42
// instructions a symbol, half of them again for codes of more than ten bits.)
//
// A VALU instruction of gfx950 may read VCC or an SGPR pair that another VALU instruction wrote
// from the third instruction after it on.

// The lane's state in a symbol loop.
struct Steps {
    BitCursor c;
    uint32_t slot;           // 5 * block in the MCU
    int32_t k;               // zig-zag index of the coefficient before the next symbol's
    uint32_t block;          // blocks completed (counting) or block of the image (writing)
    uint32_t e;              // entry of the next bits
    uint32_t end_bit, nb;    // end of the span; next restart boundary, or the end of the data
    int32_t near_w;          // from this c.w on the lane is near one of them
    __device__ __forceinline__ bool near() const { return (int32_t)c.w >= near_w; }
    // twice the number of the next symbol's table
    __device__ __forceinline__ uint32_t table(const Geometry &g) const
    {
        return __builtin_amdgcn_ubfe(g.chroma_at, slot, 3u) + (k >= 0 ? 2u : 0u);
    }
    // has the lane to be looked at before the next step?
    __device__ __forceinline__ bool due() const
    {
        const uint32_t p = c.position();
        return e == kSearchEntry || (near() && (p >= end_bit || p + entry_bits(e) > nb));
    }
    // past the entry; returns the index of its (last) symbol's coefficient
    __device__ __forceinline__ int32_t advance(const uint32_t *words, const Geometry &g)
    {
        c.advance(words, e);
        const int32_t at = k + 1 + (int32_t)entry_advance(e);
        const bool endb = at >= 63;
        slot = endb ? __builtin_amdgcn_ubfe(g.next_slot, slot, 5u) : slot;
        k = endb ? -1 : at;
        block += endb ? 1u : 0u;
        return at;
    }
};

#ifdef __AMDGCN__
// LDS byte address of what p points to
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// Parts that the written-out steps share.  What the next entry's address needs comes first; its read is
// under way while the rest is settled.  (The next stream word's read follows it: reads return in
// order, so the entry is there when at most one is left.)  vcc = the block ends, carry = a new word begins,
// t0 = the bit offset.
#define STEP_WORDS                                              \
    "s_waitcnt lgkmcnt(0)\n"                                    \
    "v_cndmask_b32 %[hi], %[hi], %[lo], %[carry]\n"             \
    "v_cndmask_b32 %[lo], %[lo], %[ahead], %[carry]\n"          \
    "v_addc_co_u32 %[w], %[m2], 0, %[w], %[carry]\n"            \
    "v_alignbit_b32 %[win], %[hi], %[lo], %[t0]\n"              \
    "v_cndmask_b32 %[slot], %[slot], %[t1], vcc\n"
// m1 = the lane is near; p = the position
#define STEP_POSITION                                           \
    "v_cmp_ge_i32 %[m1], %[w], %[nearw]\n"                      \
    "v_lshlrev_b32 %[p], 5, %[w]\n"                             \
    "v_sub_u32 %[p], %[p], %[t0]\n"
// t3, t2 = the two candidates of lookup_number
#define STEP_NUMBER                                             \
    "v_lshrrev_b32 %[t3], 22, %[win]\n"                         \
    "v_add_u32_sdwa %[t2], %[win], %[fine] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD\n"
// from t3, the number, and t0, the table
#define STEP_LOOK_UP                                            \
    "v_bfe_u32 %[t1], %[chroma], %[slot], 3\n"                  \
    "v_lshlrev_b32 %[t3], 3, %[t3]\n"                           \
    "v_addc_co_u32 %[block], %[m2], 0, %[block], vcc\n"         \
    "v_add3_u32 %[t3], %[t3], %[t1], %[t0]\n"                   \
    "ds_read_u16 %[e], %[t3]\n"                                 \
    "v_lshl_add_u32 %[t2], %[w], 2, %[aheadat]\n"               \
    "ds_read_b32 %[ahead], %[t2]\n"
// Lanes that are due are put aside: they wait for the others, and all are looked at together when no
// other lane is near.  (Spans of the same length end some twenty steps apart.  With a way out of
// the loop and back for each lane's end a span's end took a third of its time.)
#define STEP_DUE_BEGIN                                          \
    "s_mov_b64 %[all], exec\n"                                  \
    ".p2align 5\n"                                              \
    "2:\n"
#define STEP_DUE                                                \
    "v_cmp_ge_u32 %[m2], %[p], %[end]\n"                        \
    "s_waitcnt lgkmcnt(1)\n"                                    \
    "v_and_b32 %[t0], 31, %[e]\n"                               \
    "v_add_u32 %[t0], %[t0], %[p]\n"                            \
    "v_cmp_gt_u32 %[m0], %[t0], %[nb]\n"                        \
    "v_cmp_eq_u32 vcc, 0, %[e]\n"                               \
    "s_or_b64 %[m0], %[m0], %[m2]\n"                            \
    "s_and_b64 %[m0], %[m0], %[m1]\n"                           \
    "s_or_b64 %[m0], %[m0], vcc\n"                              \
    "s_andn2_b64 exec, exec, %[m0]\n"                           \
    "s_and_b64 %[m1], %[m1], exec\n"                            \
    "s_cbranch_scc1 2b\n"                                       \
    "s_mov_b64 exec, %[all]\n"                                  \
    "s_waitcnt lgkmcnt(0)\n"
// leave if a lane is near or its entry is kSearchEntry
#define STEP_NEAR                                               \
    "v_cmp_ge_i32 %[m1], %[w], %[nearw]\n"                      \
    "s_waitcnt lgkmcnt(1)\n"                                    \
    "v_cmp_eq_u32 vcc, 0, %[e]\n"                               \
    "s_or_b64 vcc, vcc, %[m1]\n"                                \
    "s_cbranch_vccz 1b\n"                                       \
    "s_waitcnt lgkmcnt(0)\n"
// (All that a step writes is marked as written early: a step reads what STEP_GIVEN lists after that.)
#define STEP_STATE                                                                                                   \
    [w] "+&v"(s.c.w), [n32] "+&v"(s.c.n32), [hi] "+&v"(s.c.hi), [lo] "+&v"(s.c.lo), [ahead] "+&v"(s.c.ahead),             \
        [win] "+&v"(s.c.win), [slot] "+&v"(s.slot), [k] "+&v"(s.k), [block] "+&v"(s.block), [e] "+&v"(s.e),               \
        [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [carry] "=&s"(carry)
#define STEP_GIVEN                                                                                                   \
    [nearw] "v"(s.near_w), [aheadat] "v"(ahead_at), [oneac] "v"(one_dc + 2u), [onedc] "v"(one_dc),                   \
        [next] "s"(g.next_slot), [chroma] "s"(g.chroma_at), [fine] "s"(0u - 63u * kFinePrefixes)
#endif

// Steps without writing, at least one, until a lane is due or the set of lanes that are near
// changes from none or to none.  Takes run entries where it may.
__device__ __forceinline__ void step_count(Steps &s, const uint32_t *words, const uint16_t *one, const uint16_t *run,
                                           const Geometry &g)
{
#ifdef __AMDGCN__
    const uint32_t ahead_at = lds_address(words) + 4u, one_dc = lds_address(one), run_dc = lds_address(run);
    uint32_t t0, t1, t2, t3;
    uint64_t m0, m1, m2, carry;
#define COUNT_ADVANCE                                           \
    "v_lshlrev_b32 %[t0], 27, %[e]\n"                           \
    "v_lshrrev_b32 %[t1], 9, %[e]\n"                            \
    "v_sub_co_u32 %[n32], %[carry], %[n32], %[t0]\n"            \
    "v_add3_u32 %[k], %[k], %[t1], 1\n"                         \
    "v_bfe_u32 %[t1], %[next], %[slot], 5\n"                    \
    "v_lshrrev_b32 %[t0], 27, %[n32]\n"                         \
    "v_cmp_lt_i32 vcc, 62, %[k]\n"                              \
    "v_cmp_lt_i32 %[m0], %[single], %[k]\n"                     \
    STEP_WORDS
    if (!wave_any(s.near())) {
        asm volatile(
            ".p2align 5\n"
            "1:\n"
            COUNT_ADVANCE
            STEP_NUMBER
            "v_cndmask_b32 %[t0], %[runac], %[oneac], %[m0]\n"
            "v_max_i32 %[t3], %[t3], %[t2]\n"
            "v_cndmask_b32 %[t0], %[t0], %[rundc], vcc\n"
            STEP_LOOK_UP
            "v_cndmask_b32 %[k], %[k], -1, vcc\n"
            STEP_NEAR
            : STEP_STATE
            : STEP_GIVEN, [runac] "v"(run_dc + 2u), [rundc] "v"(run_dc), [single] "n"(62 - kRunLead)
            : "vcc", "scc", "memory");
        if (s.near()) s.e = look_up(one, s.table(g), s.c.win);
    } else {
        uint32_t p;
        uint64_t all;
        asm volatile(
            STEP_DUE_BEGIN
            COUNT_ADVANCE
            STEP_POSITION
            STEP_NUMBER
            "s_or_b64 %[m0], %[m0], %[m1]\n"
            "v_cndmask_b32 %[t0], %[runac], %[oneac], %[m0]\n"
            "v_max_i32 %[t3], %[t3], %[t2]\n"
            "v_cndmask_b32 %[t2], %[rundc], %[onedc], %[m1]\n"
            "v_cndmask_b32 %[t0], %[t0], %[t2], vcc\n"
            STEP_LOOK_UP
            "v_cndmask_b32 %[k], %[k], -1, vcc\n"
            STEP_DUE
            : STEP_STATE, [p] "=&v"(p), [all] "=&s"(all)
            : STEP_GIVEN, [runac] "v"(run_dc + 2u), [rundc] "v"(run_dc), [single] "n"(62 - kRunLead), [end] "v"(s.end_bit), [nb] "v"(s.nb)
            : "vcc", "scc", "memory");
    }
#undef COUNT_ADVANCE
#else
    do {
        s.advance(words, g);
        s.e = look_up(s.near() || s.k > 62 - kRunLead ? one : run, s.table(g), s.c.win);
    } while (!s.due());
#endif
}

// What a writing pass needs besides.
struct WriteSteps {
    int16_t *coef;           // the image's first block
    uint32_t base;           // element for index 0: the block's, or where its DC difference goes
    uint32_t side;           // element of block 0's DC difference
    uint32_t last_block;     // of the image: a stream that runs past it goes on there, the count tells
    uint32_t over;           // bit 6: an index past its block, or bits that are no code
    int32_t iv_left, late;   // blocks left in the restart interval, less one; sign of late: a symbol after them
    bool wide;               // elements that a 32-bit byte offset does not reach
    __device__ __forceinline__ void place(const Steps &s)
    {
        const uint32_t here = min(s.block, last_block);
        base = s.k < 0 ? side + here : here << 6;
    }
};

// Steps with writing, symbol by symbol, until a lane is due or, as above, near.  Every symbol stores: ZRL and
// EOB carry no appended bits, so their value is 0, and it lands on a coefficient that they
// declare to be zero (the last of ZRL's sixteen, the last of the block for EOB).
template <bool kRestart>
__device__ __forceinline__ void step_write(Steps &s, WriteSteps &ws, const uint32_t *words, const uint16_t *one,
                                           const Geometry &g)
{
#ifdef __AMDGCN__
    const uint32_t ahead_at = lds_address(words) + 4u, one_dc = lds_address(one);
    uint32_t t0, t1, t2, t3, t4, t5, t6;
    uint64_t m0, m1, m2, carry;
// (the value's bits are taken from the window, t5 and t6, before that moves on)
#define WRITE_ADVANCE                                           \
    "v_lshlrev_b32 %[t0], 27, %[e]\n"                           \
    "v_lshrrev_b32 %[t1], 9, %[e]\n"                            \
    "v_sub_co_u32 %[n32], %[carry], %[n32], %[t0]\n"            \
    "v_sub_u32 %[t5], 0, %[e]\n"                                \
    "v_bfe_u32 %[t6], %[e], 5, 4\n"                             \
    "v_add3_u32 %[k], %[k], %[t1], 1\n"                         \
    "v_lshrrev_b32 %[t0], 27, %[n32]\n"                         \
    "v_bfe_i32 %[t5], %[win], %[t5], %[t6]\n"                   \
    "v_cmp_lt_i32 vcc, 62, %[k]\n"                              \
    "v_bfe_u32 %[t1], %[next], %[slot], 5\n"                    \
    STEP_WORDS
#define WRITE_NUMBER                                            \
    STEP_NUMBER                                                 \
    "v_cndmask_b32 %[t0], %[oneac], %[onedc], vcc\n"            \
    "v_max_i32 %[t3], %[t3], %[t2]\n"                           \
    STEP_LOOK_UP                                                \
    "v_lshlrev_b32 %[t6], %[t6], -1\n"                          \
    "v_min_i32 %[t1], 63, %[k]\n"                               \
    "v_ashrrev_i32 %[t4], 31, %[t5]\n"                          \
    "v_or_b32 %[over], %[over], %[k]\n"                         \
    "v_xor_b32 %[t6], %[t6], %[t4]\n"                           \
    "v_add_lshl_u32 %[t1], %[t1], %[base], 1\n"                 \
    "v_add3_u32 %[t4], %[t5], %[t6], 1\n"                       \
    "v_min_u32 %[t2], %[block], %[lastblock]\n"                 \
    "global_store_short %[t1], %[t4], %[coef]\n"                \
    "v_lshlrev_b32 %[base], 6, %[t2]\n"                         \
    "v_add_u32 %[t2], %[side], %[t2]\n"                         \
    "v_cndmask_b32 %[k], %[k], -1, vcc\n"                       \
    "v_cndmask_b32 %[base], %[base], %[t2], vcc\n"
#define WRITE_INTERVAL                                          \
    "v_or_b32 %[late], %[late], %[left]\n"                      \
    "v_subb_co_u32 %[left], %[m2], %[left], 0, vcc\n"
#define WRITE_STATE STEP_STATE, [t4] "=&v"(t4), [t5] "=&v"(t5), [t6] "=&v"(t6), [base] "+&v"(ws.base), [over] "+&v"(ws.over)
#define WRITE_GIVEN STEP_GIVEN, [coef] "s"(ws.coef), [lastblock] "v"(ws.last_block), [side] "v"(ws.side)
    if (!ws.wide) {
        if (!wave_any(s.near())) {
            if constexpr (kRestart)
                asm volatile(".p2align 5\n"
                             "1:\n" WRITE_ADVANCE WRITE_NUMBER WRITE_INTERVAL STEP_NEAR
                             : WRITE_STATE, [late] "+&v"(ws.late), [left] "+&v"(ws.iv_left)
                             : WRITE_GIVEN
                             : "vcc", "scc", "memory");
            else
                asm volatile(".p2align 5\n"
                             "1:\n" WRITE_ADVANCE WRITE_NUMBER STEP_NEAR
                             : WRITE_STATE
                             : WRITE_GIVEN
                             : "vcc", "scc", "memory");
        } else {
            uint32_t p;
            uint64_t all;
            if constexpr (kRestart)
                asm volatile(STEP_DUE_BEGIN WRITE_ADVANCE STEP_POSITION WRITE_NUMBER WRITE_INTERVAL STEP_DUE
                             : WRITE_STATE, [late] "+&v"(ws.late), [left] "+&v"(ws.iv_left), [p] "=&v"(p), [all] "=&s"(all)
                             : WRITE_GIVEN, [end] "v"(s.end_bit), [nb] "v"(s.nb)
                             : "vcc", "scc", "memory");
            else
                asm volatile(STEP_DUE_BEGIN WRITE_ADVANCE STEP_POSITION WRITE_NUMBER STEP_DUE
                             : WRITE_STATE, [p] "=&v"(p), [all] "=&s"(all)
                             : WRITE_GIVEN, [end] "v"(s.end_bit), [nb] "v"(s.nb)
                             : "vcc", "scc", "memory");
        }
        return;
    }
#undef WRITE_ADVANCE
#undef WRITE_NUMBER
#undef WRITE_INTERVAL
#undef WRITE_STATE
#undef WRITE_GIVEN
#endif
    do {
        const int32_t value = coefficient_value(s.c.win, entry_bits(s.e), entry_appended(s.e));
        if (kRestart) ws.late |= ws.iv_left;
        const int32_t at = s.advance(words, g);
        if (kRestart) ws.iv_left -= at >= 63 ? 1 : 0;
        ws.coef[ws.base + (uint32_t)min(at, 63)] = (int16_t)value;
        ws.over |= (uint32_t)at;
        ws.place(s);
        s.e = look_up(one, s.table(g), s.c.win);
    } while (!s.due());
}

// Decode from packed state `st` until the bit position reaches end_bit, without writing.
// words = the stream (word w at words[w]), limit_bits = end of its data.  Returns the end state;
// *nblk = blocks completed.  A symbol that does not fit before the end of the data is padding: the
// position becomes limit_bits then.  kRestart: the same before the next restart boundary (S lists
// them), where the lane steps over the boundary and goes on.
// run = the table of run entries, or that of single ones where there is none.
// (A run's last symbol, or one that is only counted, may reach past the boundary or the end of the
// data: then it did not fit.  No sound stream holds such a symbol there, with ten bits and more left.)
template <bool kRestart, typename Shared>
__device__ __forceinline__ uint32_t count_span(const Shared &S, const uint32_t *words, const uint16_t *run,
                                               const Geometry &g, uint32_t st, uint32_t end_bit, uint32_t limit_bits,
                                               uint32_t *nblk)
{
    const uint16_t *one = S.tab.one;
    uint32_t p = st >> 9;
    Steps s;
    s.slot = slot_of_block((st >> 6) & 7u);
    s.k = (int32_t)(st & 63u) - 1;
    s.block = 0;
    s.end_bit = end_bit;
    s.nb = limit_bits;
    if constexpr (kRestart) s.nb = boundary_from(S, (p + 7u) >> 3, limit_bits);
    // far away, all symbols of a run but the last end before the span does
    auto near_from = [&]() { return ((int32_t)(min(s.end_bit, s.nb) - kRunLeadBits - 1u) >> 5) + 1; };
    s.near_w = near_from();
    s.c.start(words, p);
    s.e = look_up(s.near() || s.k > 62 - kRunLead ? one : run, s.table(g), s.c.win);
    for (;;) {
        if (s.e == kSearchEntry) s.e = lookup_by_search(S.tab, s.table(g) >> 1, s.c.win);
        if (s.near()) {
            p = s.c.position();
            while (p > s.nb || (p < end_bit && p + entry_bits(s.e) > s.nb)) {
                if (!kRestart || s.nb >= limit_bits) {
                    p = limit_bits;
                    break;
                }
                if constexpr (kRestart) {
                    p = s.nb;
                    s.slot = 0;
                    s.k = -1;
                    s.nb = boundary_from(S, (p >> 3) + 1u, limit_bits);
                    s.near_w = near_from();
                    s.c.start(words, p);
                    s.e = look_up(one, 0, s.c.win);
                    if (s.e == kSearchEntry) s.e = lookup_by_search(S.tab, 0, s.c.win);
                }
            }
            if (p >= end_bit) break;
        }
        step_count(s, words, one, run, g);
    }
    *nblk = s.block;
    return pack_state(p, block_of_slot(s.slot), (uint32_t)(s.k + 1));
}

// The same with writing: single symbols, exact at every one.  DC *differences* go to the image's
// side array, one entry per block (dc_prefix turns them into values and puts those into the
// blocks).  Refuses (wc->bad) what a sound stream cannot hold.
// Where the end of the span is the end of its restart interval, kRestart = false and limit_bits =
// end_bit do.
template <bool kRestart, typename Shared>
__device__ __forceinline__ uint32_t write_span(const Shared &S, const uint32_t *words, const Geometry &g, uint32_t st,
                                               uint32_t end_bit, uint32_t limit_bits, uint32_t *nblk, WriteCtx *wc)
{
    const uint16_t *one = S.tab.one;
    uint32_t p = st >> 9;
    int32_t broken = 0;
    Steps s;
    s.slot = slot_of_block((st >> 6) & 7u);
    s.k = (int32_t)(st & 63u) - 1;
    s.block = wc->block;
    s.end_bit = end_bit;
    s.nb = limit_bits;
    if constexpr (kRestart) s.nb = boundary_from(S, (p + 7u) >> 3, limit_bits);
    // far away, any symbol ends before the span does (31 bits at most)
    auto near_from = [&]() { return ((int32_t)(min(s.end_bit, s.nb) - 32u) >> 5) + 1; };
    s.near_w = near_from();
    WriteSteps ws;
    ws.coef = wc->coef;
    ws.side = wc->side_rel;
    ws.last_block = g.n_blocks - 1u;
    ws.over = 0;
    ws.iv_left = kRestart ? wc->iv_rem - 1 : 0;
    ws.late = 0;
    ws.wide = (((uint64_t)wc->side_rel + g.n_blocks) >> 31) != 0 || ((uint64_t)g.n_blocks >> 25) != 0;
    ws.place(s);
    s.c.start(words, p);
    s.e = look_up(one, s.table(g), s.c.win);
    for (;;) {
        if (s.e == kSearchEntry) s.e = lookup_by_search(S.tab, s.table(g) >> 1, s.c.win);
        if (s.near()) {
            p = s.c.position();
            while (p < end_bit && p + entry_bits(s.e) > s.nb) {
                if (!kRestart || s.nb >= limit_bits) {
                    // what is left is padding: fewer than eight bits, between MCUs
                    if (s.slot != 0 || s.k >= 0 || limit_bits - p >= 8) broken = 1;
                    p = limit_bits;
                    break;
                }
                if constexpr (kRestart) {
                    // a boundary comes between MCUs, behind fewer than eight padding bits,
                    // and after a whole interval (or right where one has just begun)
                    if (s.slot != 0 || s.k >= 0 || s.nb - p >= 8 || g.ri_blocks == 0 ||
                        (ws.iv_left != -1 && ws.iv_left != (int32_t)g.ri_blocks - 1))
                        broken = 1;
                    ws.iv_left = (int32_t)g.ri_blocks - 1;
                    p = s.nb;
                    s.slot = 0;
                    s.k = -1;
                    s.nb = boundary_from(S, (p >> 3) + 1u, limit_bits);
                    s.near_w = near_from();
                    ws.place(s);
                    s.c.start(words, p);
                    s.e = look_up(one, 0, s.c.win);
                    if (s.e == kSearchEntry) s.e = lookup_by_search(S.tab, 0, s.c.win);
                }
            }
            if (p >= end_bit) break;
        }
        if (s.e == kInvalidDcEntry) broken = 1;
        step_write<kRestart>(s, ws, words, one, g);
    }
#ifdef __AMDGCN__
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores that the compiler has not seen
#endif
    wc->bad |= broken | (ws.late < 0 ? 1 : 0) | (int32_t)((ws.over >> 6) & 1u);
    *nblk = s.block - wc->block;
    return pack_state(p, block_of_slot(s.slot), (uint32_t)(s.k + 1));
}

// Zeros over the blocks [lo, hi) of an image whose coefficients begin at coef, in 16-byte units
// first, first + step, ... of the range's eight per block.  Nothing clears the coefficient
// workspace before the decoder runs, and the writing passes store only the coefficients that
// symbols name: a workgroup begins with zeros over all blocks that it is to decode, in whole
// 128-byte lines, and has barriers before its first coefficient.  (Stored by each lane over its own
// blocks, right before these, they took a tenth of the time for long intervals.)  Out of line: it
// must not add to the registers of the symbol loops.
__device__ __attribute__((noinline)) void zero_blocks(int16_t *coef, uint32_t lo, uint32_t hi, uint32_t first,
                                                      uint32_t step)
{
    uint4 *units = reinterpret_cast<uint4 *>(coef);  // eight to a block
    for (uint32_t u = lo * 8u + first; u < hi * 8u; u += step) units[u] = make_uint4(0, 0, 0, 0);
}

// DC differences -> DC values (T.81 F.2.2.1) for blocks [lo, hi) of the image, by the whole
// workgroup.  The writing passes leave the differences in the image's side array (one int16 per
// block, so both walks below read a few cache lines instead of one line per block); the values go
// into the blocks.  Each lane takes a contiguous run of blocks, sums its differences per component (a
// sum restarts where a restart interval begins), a segmented scan over the lanes carries the
// running values in, and a second walk writes them.  carry[] = running value of each
// component before block lo; on return, after block hi - 1.  All lanes must call.
// Blocks are read eight at a time so that the loads do not wait for one another.
struct DcWalk {
    uint32_t in_mcu, in_iv;  // position of the block in its MCU and in its restart interval
    __device__ inline void start(const Geometry &g, uint32_t block)
    {
        in_mcu = block % g.bpm;
        in_iv = g.ri_blocks ? block % g.ri_blocks : block;
    }
    // the first block of each component in the first MCU of an interval restarts DC prediction
    __device__ inline bool restarts(const Geometry &g) const
    {
        return in_iv == 0 || (in_iv >= g.n_luma && in_iv < g.bpm);
    }
    __device__ inline uint32_t comp(const Geometry &g) const { return comp_of_block(g, in_mcu); }
    __device__ inline void next(const Geometry &g)
    {
        in_mcu = in_mcu + 1u == g.bpm ? 0u : in_mcu + 1u;
        in_iv++;
        if (g.ri_blocks && in_iv == g.ri_blocks) in_iv = 0;
    }
};

__device__ inline void dc_prefix(int32_t *scan_val, int32_t *scan_flag, const Geometry &g, int16_t *coef,
                                 const int16_t *side, uint32_t lo, uint32_t hi, int32_t carry[3])
{
    __syncthreads();  // the stores of every lane (zeros, coefficients, differences) are done and visible
    const uint32_t n = hi > lo ? hi - lo : 0u;
    const uint32_t per = (n + kT - 1) / kT;
    const uint32_t a = min(lo + threadIdx.x * per, hi), b = min(a + per, hi);
    int32_t s0 = 0, s1 = 0, s2 = 0, r0 = 0, r1 = 0, r2 = 0;
    DcWalk wk;
    wk.start(g, a);
    for (uint32_t i = a; i < b; i += 8) {
        int32_t d[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; u++) d[u] = side[min(i + u, b - 1)];
#pragma unroll
        for (uint32_t u = 0; u < 8; u++) {
            if (i + u < b) {
                const uint32_t c = wk.comp(g);
                const bool rst = wk.restarts(g);
                if (c == 0) { s0 = (rst ? 0 : s0) + d[u]; r0 |= rst; }
                else if (c == 1) { s1 = (rst ? 0 : s1) + d[u]; r1 |= rst; }
                else { s2 = (rst ? 0 : s2) + d[u]; r2 |= rst; }
                wk.next(g);
            }
        }
    }
    int32_t out;
    int32_t c0 = block_seg_excl_scan(s0, r0, carry[0], scan_val, scan_flag, &out);
    carry[0] = out;
    int32_t c1 = block_seg_excl_scan(s1, r1, carry[1], scan_val, scan_flag, &out);
    carry[1] = out;
    int32_t c2 = block_seg_excl_scan(s2, r2, carry[2], scan_val, scan_flag, &out);
    carry[2] = out;
    wk.start(g, a);
    for (uint32_t i = a; i < b; i += 8) {
        int32_t d[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; u++) d[u] = side[min(i + u, b - 1)];
#pragma unroll
        for (uint32_t u = 0; u < 8; u++) {
            if (i + u < b) {
                const uint32_t c = wk.comp(g);
                const bool rst = wk.restarts(g);
                int32_t v;
                if (c == 0) { c0 = (rst ? 0 : c0) + d[u]; v = c0; }
                else if (c == 1) { c1 = (rst ? 0 : c1) + d[u]; v = c1; }
                else { c2 = (rst ? 0 : c2) + d[u]; v = c2; }
                coef[(size_t)(i + u) * 64] = (int16_t)v;
                wk.next(g);
            }
        }
    }
}

__device__ inline uint32_t load_byte(const uint8_t *p) { return *p; }

// binary search: largest i with key(i) <= x over records sorted by a uint32 field
template <typename F>
__device__ inline int find_image(int n, uint32_t x, F key)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (key(mid) <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The same by a whole wave (all lanes must call), in two loads that wait for each other instead
// of one for every halving: a kernel of many images begins 2 to 3 us earlier.
template <typename F>
__device__ inline int find_image_wave(int n, uint32_t x, F key)
{
    const int lane = threadIdx.x & 63, s = (n + 63) / 64;
    if (s > 64) return find_image(n, x, key);
    int lo = 0;
    if (s > 1) lo = s * max(0, __popcll(__ballot(lane * s < n && key(min(lane * s, n - 1)) <= x)) - 1);
    const int i = lo + lane;
    return lo + max(0, __popcll(__ballot((s == 1 || lane < s) && i < n && key(min(i, n - 1)) <= x)) - 1);
}

// Which raw bytes of one 16-byte piece are entropy-coded data (keep) and which are the
// code byte of an RSTn marker (bound).  prev = the byte before the piece, next = the byte
// after it.  Bytes outside [cs, ce) are neither.  A byte after FF is stuffing or a marker
// code; FF itself is data only before 00.
__device__ inline void classify16(const uint4 v, uint32_t prev, uint32_t nextb, int32_t plo,
                                  int32_t cs, int32_t ce, uint32_t *keep, uint32_t *bound,
                                  uint32_t *last, int32_t *bad)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t k = 0, b = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const uint32_t cur = (w[i >> 2] >> (8 * (i & 3))) & 255u;
        const uint32_t nxt = i < 15 ? (w[(i + 1) >> 2] >> (8 * ((i + 1) & 3))) & 255u : nextb;
        const int32_t pos = plo + i;
        const bool inside = pos >= cs && pos < ce;
        const bool kp = cur == 0xFFu ? nxt == 0u : prev != 0xFFu;
        if (inside && kp) k |= 1u << i;
        if (inside && prev == 0xFFu && cur != 0u) {
            if (cur >= 0xD0u && cur <= 0xD7u) b |= 1u << i;
            else if (cur != 0xFFu) *bad = 1;  // a marker that may not occur inside a scan
        }
        prev = cur;
    }
    *keep = k;
    *bound = b;
    *last = prev;
}

// Packs the bytes that staging keeps into big-endian words, a lane its own piece of the stream.  A lane
// puts the words whose last byte is its own, with zeros for bytes of the lanes before; its last
// bytes, fewer than four, are ORed into their word after a barrier.  Words without stuffing or
// markers in any lane go through whole.  (A byte at a time took 25 of the 177 us that a workgroup
// spends on a 12 KB restart interval, three less now.)
struct BytePacker {
    uint32_t word, n;  // word of the destination, and how many of its bytes precede
    uint32_t acc = 0;  // the last n bytes, in its low bits
    __device__ BytePacker(uint32_t byte) : word(byte >> 2), n(byte & 3u) {}
    __device__ uint32_t at() const { return 4u * word + n; }
    // the bytes of w (the lowest first) that are set in keep4; put(index, word) stores
    template <typename Put>
    __device__ __forceinline__ void add(uint32_t w, uint32_t keep4, Put put)
    {
        if (!wave_any(keep4 != 15u)) {
            const uint32_t v = __builtin_bswap32(w);
            put(word++, __builtin_amdgcn_alignbit(acc, v, 8u * n));
            acc = v;
            return;
        }
        uint32_t c = 0, more = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const bool kept = ((keep4 >> i) & 1u) != 0;
            c = kept ? (c << 8) | ((w >> (8 * i)) & 255u) : c;
            more += kept ? 1u : 0u;
        }
        const uint64_t both = ((uint64_t)acc << (8u * more)) | c;
        n += more;
        if (n >= 4u) {
            n -= 4u;
            put(word++, (uint32_t)(both >> (8u * n)));
        }
        acc = (uint32_t)both;
    }
    __device__ uint32_t rest() const { return acc << (32u - 8u * n); }  // (n != 0)
};

__device__ inline void stream_geometry(Geometry &g, const ImageRec &R)
{
    g.bpm = R.blocks_per_mcu;
    g.n_luma = (uint32_t)(luma_h(R.sampling) * luma_v(R.sampling));
    g.ri_blocks = 0;
    g.set_slots();
    g.n_blocks = R.n_blocks;
}

// image of stream window wg: the last one whose first window does not exceed it (images without
// stream windows share their number with the next one that has some)
__device__ inline int image_of_stream(const ImageRec *recs, int n_images, uint32_t wg)
{
    return find_image_wave(n_images, wg, [&](int i) { return recs[i].stream0; });
}

// DC differences -> DC values of the blocks whose DC was decoded in stream window wg (all lanes of the
// workgroup must call).
__device__ inline void finish_window(const ImageRec *__restrict__ recs, int n_images, uint32_t wg,
                                     const uint32_t *__restrict__ retry, const StreamWindow *__restrict__ windows,
                                     int16_t *__restrict__ coef_all, uint32_t side_off, uint32_t *scan_a, int32_t *dc_val,
                                     int32_t *dc_flag)
{
    const int img = image_of_stream(recs, n_images, wg);
    const ImageRec &R = recs[img];
    const uint32_t w = wg - R.stream0;
    if (w >= R.n_streams || R.status != PREP_OK || retry[img] != 0) return;
    const StreamWindow *W = windows + R.stream0;
    if (W[w].dc_hi <= W[w].dc_lo) return;
    uint32_t before[3] = {0, 0, 0};
    for (uint32_t i = threadIdx.x; i < w; i += kT)
#pragma unroll
        for (int c = 0; c < 3; c++) before[c] += (uint32_t)W[i].dc_sum[c];
    int32_t carry[3];
#pragma unroll
    for (int c = 0; c < 3; c++) carry[c] = (int32_t)block_sum(before[c], scan_a);
    Geometry g;
    stream_geometry(g, R);
    int16_t *coef = coef_all + (size_t)R.coef_block0 * 64;
    dc_prefix(dc_val, dc_flag, g, coef, coef + (side_off + R.coef_block0 - R.coef_block0 * 64u), W[w].dc_lo, W[w].dc_hi, carry);
}

}  // namespace

// ---- kernel 1: restart markers per window -----------------------------------
// window w of an image = raw bytes [w*window_bytes, (w+1)*window_bytes) of its
// entropy-coded segment.  cnt = RSTn markers whose FF byte lies in the window,
// first = offset (from the segment start) of the first such FF byte.
// data_end[image] arrives as the length that the host gave the segment (up to the file's last
// EOI marker, which it finds from the file's end) and leaves as the offset of the first EOI
// marker in it: FF D9 cannot occur inside entropy-coded data (T.81 F.1.2.3), so where a file
// goes on after its image (a second image, a preview) the data end there.
// Workgroups from n_windows on do something else: workgroup n_windows + 4 (kTableParts s + p) + t
// expands part p of Huffman table t of image table_rep[s] into slot s of `tables`.
__global__ __launch_bounds__(kDecodeThreads) void scan_restart_markers(
    const uint8_t *__restrict__ bits, const ImageRec *__restrict__ recs, int n_images,
    uint32_t n_windows, uint32_t window_bytes, uint32_t *__restrict__ win_count,
    uint32_t *__restrict__ win_first, uint32_t *__restrict__ data_end, uint32_t *__restrict__ retry,
    int32_t *__restrict__ status, const uint32_t *__restrict__ table_rep, bool runs, uint4 *__restrict__ tables)
{
    __shared__ uint32_t s_cnt[kT / 64], s_first[kT / 64];
    const uint32_t wg = blockIdx.x;
    if (wg >= n_windows) {
        const uint32_t id = wg - n_windows, slot = id / (4u * kTableParts);
        const ImageRec &I = recs[table_rep[slot]];
        expand_table(bits + I.file_off, I, (int)(id & 3u), id / 4u % kTableParts, runs,
                     reinterpret_cast<HuffTables *>(tables) + slot);
        return;
    }
    const int img = find_image_wave(n_images, wg, [&](int i) { return recs[i].window0; });
    const ImageRec &R = recs[img];
    const uint32_t w = wg - R.window0;
    // the per-image verdict starts as the host parser's; the decoder may lower it
    if (w == 0 && threadIdx.x == 0) {
        status[img] = R.status;
        retry[img] = 0;
    }
    uint32_t cnt = 0, first = kNoMarker, eoi = kNoMarker;
    if (R.status == PREP_OK && w < R.n_windows) {
        const bool count_rst = R.restart_interval != 0;
        const uint8_t *seg = bits + R.file_off + R.entropy_rel;
        const int32_t lo = (int32_t)(w * window_bytes);
        const int32_t hi = (int32_t)min(w * window_bytes + window_bytes, R.entropy_len);
        // 16-byte aligned parts that cover [lo, hi), dealt to the lanes in turn; a part that
        // begins before lo reaches at most 15 bytes back, into the file's headers
        const int32_t a0 = lo - (int32_t)((uintptr_t)(seg + lo) & 15u);
        for (int32_t plo = a0 + 16 * (int32_t)threadIdx.x; plo < hi; plo += 16 * kT) {
            const uint4 v = *reinterpret_cast<const uint4 *>(seg + plo);
            // the byte after the last one of the segment is the EOI marker's FF
            const uint32_t after = load_byte(seg + min(plo + 16, (int32_t)R.entropy_len));
            const uint32_t wv[5] = {v.x, v.y, v.z, v.w, after};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                // a byte FF before one of D0 to DF, four at a time: a zero byte here
                const uint32_t next = __builtin_amdgcn_alignbit(wv[e + 1], wv[e], 8u);
                const uint32_t z = ~wv[e] | ((next & 0xF0F0F0F0u) ^ 0xD0D0D0D0u);
                if (((z - 0x01010101u) & ~z & 0x80808080u) == 0) continue;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const uint32_t cur = (wv[e] >> (8 * i)) & 255u, nxt = (next >> (8 * i)) & 255u;
                    const int32_t pos = plo + 4 * e + i;
                    if (cur == 0xFFu && nxt >= 0xD0u && nxt <= 0xD9u && nxt != 0xD8u && pos >= lo && pos < hi) {
                        if (nxt == 0xD9u) {
                            eoi = min(eoi, (uint32_t)pos);
                        } else if (count_rst) {
                            cnt++;
                            first = min(first, (uint32_t)pos);
                        }
                    }
                }
            }
        }
        if (eoi != kNoMarker) atomicMin(&data_end[img], eoi);
    }
    // workgroup reduction
    for (int d = 32; d >= 1; d >>= 1) {
        cnt += __shfl_xor(cnt, d, 64);
        first = min(first, (uint32_t)__shfl_xor(first, d, 64));
    }
    if ((threadIdx.x & 63) == 0) { s_cnt[threadIdx.x >> 6] = cnt; s_first[threadIdx.x >> 6] = first; }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t c = 0, f = kNoMarker;
        for (int i = 0; i < kT / 64; i++) { c += s_cnt[i]; f = min(f, s_first[i]); }
        win_count[wg] = c;
        win_first[wg] = f;
    }
}

// ---- kernel 2: the decoder -----------------------------------------------------
// kHyp: the variant for calls with little data, whose workgroups own a few restart intervals
// each (small windows).  Inside a restart interval the state at a subsequence border is not
// known; what keeps iteration slow there is the block's place in the MCU (which tables come
// next), while bit position and zig-zag index fall into step within a block or two.  So every
// subsequence is decoded once from each place-in-MCU hypothesis by a lane of its own (the chip
// is idle otherwise), and once more from the end states those lanes reached in the subsequence
// before; the true chain then only picks, link by link, the candidate that it equals.
// Workgroups from n_windows on finish the stream windows that write_streams wrote, one each: they
// share nothing with the others (an image is decoded in windows or here), and a kernel of their own
// costs a call with one image 5 us.
template <bool kHyp, bool kRuns>
__global__ __launch_bounds__(kDecodeThreads, kRuns ? 3 : 4) void decode_entropy(
    const uint8_t *__restrict__ bits, const ImageRec *__restrict__ recs, int n_images,
    const uint32_t *__restrict__ win_count, const uint32_t *__restrict__ win_first,
    const uint32_t *__restrict__ data_end, const uint32_t *__restrict__ retry, int16_t *__restrict__ coef_all,
    uint32_t side_off, int32_t *__restrict__ status, const uint4 *__restrict__ tables, uint32_t hyp_span_bits,
    uint32_t n_windows, const StreamWindow *__restrict__ windows)
{
    __shared__ DecodeShared<kHyp, kRuns> S;
    static_assert(kHyp || workgroups_by_lds(sizeof(S)) >= (kRuns ? 3u : 4u), "as many as the launch bounds say");
    const uint16_t *const runs = run_entries(S.tab);
    const int tid = threadIdx.x;
    const uint32_t wg = blockIdx.x;
    if (wg >= n_windows) {
        finish_window(recs, n_images, wg - n_windows, retry, windows, coef_all, side_off, S.scan_a, S.dc_val, S.dc_flag);
        return;
    }
    const int img = find_image_wave(n_images, wg, [&](int i) { return recs[i].window0; });
    const ImageRec &R = recs[img];
    const uint32_t w = wg - R.window0;
    if (R.status != PREP_OK || w >= R.n_windows) return;
    if (R.n_streams != 0 && retry[img] == 0) return;  // decoded by write_streams

    Geometry g;
    g.bpm = R.blocks_per_mcu;
    g.n_luma = (uint32_t)(luma_h(R.sampling) * luma_v(R.sampling));
    g.ri_blocks = (uint32_t)R.restart_interval * g.bpm;
    g.set_slots();
    g.n_blocks = R.n_blocks;

    // ---- which part of the stream is ours -------------------------------------
    // window 0 starts at the segment start; window w > 0 starts after the first
    // marker of its window, if it has one, and runs to the first marker of the
    // next window that has one.
    // the entropy-coded data end at the segment's first EOI marker (found by the scan kernel)
    const uint32_t data_len = min(R.entropy_len, data_end[img]);
    uint32_t range_lo = 0, range_hi = data_len, block0 = 0, block_end = R.n_blocks;
    uint32_t marker_base = 0;  // number, within the image, of the first restart marker at or after cs
    bool first_marker_ok = true;
    {
        const uint32_t *wc = win_count + R.window0, *wf = win_first + R.window0;
        uint32_t my_first = w == 0 ? 0u : wf[w];
        if (w != 0 && (my_first == kNoMarker || my_first >= data_len)) return;  // uniform over the workgroup
        uint32_t before = 0, next_first = kNoMarker, next_w = kNoMarker;
        for (uint32_t i = tid; i < w; i += kT) before += wc[i];
        for (uint32_t i = w + 1 + tid; i < R.n_windows; i += kT)
            if (wf[i] != kNoMarker) { next_w = i; next_first = wf[i]; break; }
        for (int d = 32; d >= 1; d >>= 1) {
            before += __shfl_xor(before, d, 64);
            uint32_t ow = __shfl_xor(next_w, d, 64), of = __shfl_xor(next_first, d, 64);
            if (ow < next_w) { next_w = ow; next_first = of; }
        }
        if ((tid & 63) == 0) {
            S.scan_a[tid >> 6] = before;
            S.dc_val[tid >> 6] = (int32_t)next_w;
            S.dc_flag[tid >> 6] = (int32_t)next_first;
        }
        __syncthreads();
        before = 0;
        next_w = kNoMarker;
        for (int i = 0; i < kT / 64; i++) {
            before += S.scan_a[i];
            if ((uint32_t)S.dc_val[i] < next_w) {
                next_w = (uint32_t)S.dc_val[i];
                next_first = (uint32_t)S.dc_flag[i];
            }
        }
        __syncthreads();
        if (next_w != kNoMarker && next_first >= data_len) next_w = kNoMarker;  // (a marker of what follows the image)
        if (w != 0) {
            range_lo = my_first + 2;
            block0 = (before + 1) * g.ri_blocks;  // markers before ours + ours = intervals done
            marker_base = before + 1;
            // our marker is number `before` of the image, and markers count modulo 8 from RST0
            // (T.81 E.2.4, B.2.1); the markers inside the run are checked where they are staged
            first_marker_ok = ((load_byte(bits + R.file_off + R.entropy_rel + my_first + 1) ^ before) & 7u) == 0;
        }
        if (next_w != kNoMarker) {
            range_hi = next_first;
            // markers up to and including the first one of window next_w
            uint32_t upto = 0;
            for (uint32_t i = tid; i < next_w; i += kT) upto += wc[i];
            upto = block_sum(upto, S.scan_a);
            block_end = (upto + 1) * g.ri_blocks;
        }
    }
    if (block0 >= R.n_blocks || block_end > R.n_blocks || range_lo > range_hi || !first_marker_ok) {
        if (tid == 0) atomicMin(&status[img], (int32_t)PREP_E_CORRUPT);
        return;
    }

    const uint8_t *file = bits + R.file_off;
    if (R.table_slot != kNoTableSlot) {
        // the tables were expanded once for the batch: copy them
        load_tables(S.tab, tables, R.table_slot);
        __syncthreads();
    } else {
        build_tables(S.tab, file, R);
        if constexpr (kRuns) build_runs(S.tab);
    }

    const uint8_t *seg = file + R.entropy_rel;
    int16_t *coef = coef_all + (size_t)R.coef_block0 * 64;
    // DC differences of this image's blocks: the side array begins side_off elements after the
    // first coefficient of the workspace, one entry per block
    const uint32_t side_rel = side_off + R.coef_block0 - R.coef_block0 * 64u;
    // raw offsets are signed: the aligned span of the first chunk may begin a few bytes
    // before the segment (inside the file's headers)
    const int32_t seg_len = (int32_t)data_len;
    const int32_t rhi = (int32_t)range_hi;
    int32_t cs = (int32_t)range_lo;      // raw offset where the next chunk starts
    uint32_t st0 = pack_state(0, 0, 0);  // true state at the start of the chunk
    uint32_t block_base = block0;
    int32_t dc_carry[3] = {0, 0, 0};
    int32_t bad = 0;

    const uint32_t max_chunks = (range_hi - range_lo) / 64u + 2;
    for (uint32_t iter = 0; iter < max_chunks && cs < rhi; iter++) {
        // what a chunk hands on to the next came through LDS: the same in every lane, but the compiler does
        // not know, and of the 128 vector registers of the variant for short intervals none are spare
        cs = __builtin_amdgcn_readfirstlane(cs);
        st0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)st0);
        block_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)block_base);
        marker_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)marker_base);
#pragma unroll
        for (int c = 0; c < 3; c++) dc_carry[c] = __builtin_amdgcn_readfirstlane(dc_carry[c]);
        // ---- stage: destuff raw bytes [cs, ce) into S.clean --------------------------
        // lanes own 64-byte pieces (four 16-byte parts) of the 16-byte aligned span that
        // contains cs
        const int32_t mis = (int32_t)((uintptr_t)(seg + cs) & 15u);
        const int32_t a0 = cs - mis;
        const int32_t ce = min(a0 + (int32_t)kChunkRaw, rhi);
        const bool last = ce == rhi;
        __syncthreads();
        for (int i = tid; i < kMaskWords; i += kT) S.bmask[i] = 0;
        const int32_t my_lo = a0 + tid * 64;  // raw offset of my first byte
        // 16-byte parts are loaded whether or not they still overlap [cs, ce] (what lies
        // outside is not looked at), from an address clamped to the part that holds ce, so
        // that the loads of a piece do not wait for one another.  Such a load is aligned
        // and holds at least one byte of the file, so it stays inside the file's last page.
        const int32_t last_part = a0 + ((ce - a0) & ~15);
        uint4 v[4];
#pragma unroll
        for (int k = 0; k < 4; k++)
            v[k] = *reinterpret_cast<const uint4 *>(seg + min(my_lo + 16 * k, last_part));
        unsigned long long keep = 0, bound = 0;
        {
            // the byte before my piece and the byte after each 16-byte part, for the FF xx
            // pairs that straddle; past the segment comes the FF of the EOI marker
            const uint32_t after = load_byte(seg + min(my_lo + 64, ce));
            uint32_t prev = 0;
            if (my_lo > cs && my_lo <= ce) prev = load_byte(seg + my_lo - 1);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int32_t plo = my_lo + 16 * k;
                uint32_t kp = 0, bd = 0;
                // a part is looked at only if it overlaps [cs, ce]: the byte at ce (the FF of
                // the marker that ends the run) is examined, not consumed
                if (plo <= ce) {
                    uint32_t nextb = k < 3 ? (v[(k + 1) & 3].x & 255u) : after;
                    if (!(plo + 16 < seg_len && plo + 16 <= ce)) nextb = 0xFFu;
                    classify16(v[k], prev, nextb, plo, cs, ce, &kp, &bd, &prev, &bad);
                } else {
                    prev = 0;
                }
                keep |= (unsigned long long)kp << (16 * k);
                bound |= (unsigned long long)bd << (16 * k);
            }
        }
        // clean offsets (low half) and boundary ranks (high half) in one scan
        uint32_t totals;
        const uint32_t my_pre = block_excl_scan((uint32_t)__popcll(keep) | ((uint32_t)__popcll(bound) << 16),
                                                S.scan_a, &totals);
        const uint32_t clean_len = totals & 0xFFFFu, nbnd = totals >> 16;
        const uint32_t my_off = my_pre & 0xFFFFu;
        if (iter == 0) zero_blocks(coef, block0, block_end, (uint32_t)tid, kT);  // (behind the loads)
        S.keep_off[tid] = my_off;
        if (tid == 0) S.keep_off[kT] = clean_len;
        // Which of the two passes will decode the chunk is known now.  Intervals 0..n_iv-1 of
        // the chunk end inside it: the first runs from the chunk's start state to the first
        // listed start, interval k > 0 between listed starts k-1 and k, and in the last chunk
        // one more runs to the end of the data.
        const uint32_t n_iv = last ? nbnd + 1 : nbnd;
        // (the variant for small calls finds the states inside restart intervals by hypotheses)
        const bool by_hypotheses = kHyp && g.ri_blocks != 0;
        const bool short_intervals = !by_hypotheses && g.ri_blocks != 0 && n_iv >= 1 &&
                                     nbnd <= (uint32_t)kMaxBoundaries && clean_len <= kShortInterval * (nbnd + 1);
        // the short-interval pass reads the stream without pad words (its lanes start anywhere)
        const uint32_t pad_shift = short_intervals ? 31u : (uint32_t)kPadShift;
        if constexpr (!kHyp)
            if (!short_intervals) S.keep[tid] = keep;
        // zeros behind the data: its last word is put together with OR, and lookups near the
        // end read a few words past it
        {
            // (a run of array entries: in the subsequence passes it takes in the rows' last words,
            // the copies, among them the copy of the data's last, partly written word)
            const uint32_t wd = clean_len >> 2, first = wd + (wd >> pad_shift);
            const uint32_t from = !short_intervals && (wd & 15u) == 0 && wd != 0 ? first - 1u : first;
            if (tid < 14) S.clean[from + (uint32_t)tid] = 0;
        }
        {
            BytePacker pack(my_off);
            uint32_t rank = my_pre >> 16;
            auto put = [&](uint32_t wq, uint32_t word) {
                const uint32_t at = wq + (wq >> pad_shift);
                S.clean[at] = word;
                // the first word of a subsequence is also the last of the row before
                if (!short_intervals && (wq & 15u) == 0 && wq != 0) S.clean[at - 1u] = word;
            };
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t kp = (uint32_t)(keep >> (16 * k)) & 0xFFFFu;
                const uint32_t bd = (uint32_t)(bound >> (16 * k)) & 0xFFFFu;
                if ((kp | bd) == 0) continue;
                const uint32_t wv[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t keep4 = (kp >> (4 * e)) & 15u;
                    uint32_t marks = (bd >> (4 * e)) & 15u;
                    while (marks != 0) {
                        const uint32_t i = (uint32_t)__builtin_ctz(marks);
                        marks &= marks - 1u;
                        const uint32_t o = pack.at() + (uint32_t)__popcll(keep4 & ((1u << i) - 1u));
                        // marker number marker_base + rank of the image must be RST((that) mod 8)
                        if ((((wv[e] >> (8 * i)) ^ (marker_base + rank)) & 7u) != 0) bad = 1;
                        atomicOr(&S.bmask[o >> 5], 1u << (o & 31));
                        if (short_intervals) S.bpos[rank] = (uint16_t)o;  // (at most kMaxBoundaries then)
                        // raw offset just after the last marker of the chunk: where a chunk of
                        // whole intervals would resume
                        if (rank + 1 == nbnd) S.bcast[2] = (uint32_t)(my_lo + 16 * k + 4 * e + (int32_t)i + 1);
                        rank++;
                    }
                    pack.add(wv[e], keep4, put);
                }
            }
            __syncthreads();  // (the words, and the zeros behind the data, are there)
            if (pack.n != 0) {
                const uint32_t wq = pack.word, at = wq + (wq >> pad_shift);
                atomicOr(&S.clean[at], pack.rest());
                if (!short_intervals && (wq & 15u) == 0 && wq != 0) atomicOr(&S.clean[at - 1u], pack.rest());
            }
        }
        __syncthreads();
        {
            // first interval start at or after each lane's subsequence: suffix minimum
            unsigned long long m = ((unsigned long long)S.bmask[2 * tid + 1] << 32) | S.bmask[2 * tid];
            uint32_t mine = m ? (uint32_t)tid * 64u + (uint32_t)__builtin_ctzll(m) : kNoMarker;
            const int lane = tid & 63, wave = tid >> 6;
            for (int d = 1; d < 64; d <<= 1) {
                uint32_t o = __shfl_down(mine, d, 64);
                if (lane + d < 64) mine = min(mine, o);
            }
            if (lane == 0) S.scan_a[wave] = mine;
            __syncthreads();
            uint32_t later = kNoMarker;
            for (int ww = wave + 1; ww < kT / 64; ww++) later = min(later, S.scan_a[ww]);
            S.next_boundary[tid] = min(mine, later);
            if (tid == 0) S.next_boundary[kT] = kNoMarker;
        }
        __syncthreads();

        const uint32_t limit_bits = clean_len * 8u;
        WriteCtx wc;
        wc.coef = coef;
        wc.side_rel = side_rel;
        wc.bad = 0;

        // ---- short intervals: one lane per restart interval, one pass -----------------
        // A decoding lane is bound by the latency of its own dependent instructions, and a
        // wave takes as long as its slowest lane whatever the number of busy lanes:
        // consecutive intervals go to consecutive lanes, so that they fill as few waves as
        // possible and the other waves of the workgroup leave their SIMDs to other workgroups.
        if (short_intervals) {
            const uint32_t rem0 = g.ri_blocks - block_base % g.ri_blocks;  // blocks left in interval 0
            for (uint32_t k = (uint32_t)tid; k < n_iv; k += kT) {
                const uint32_t start = k ? pack_state((uint32_t)S.bpos[k - 1] * 8u, 0, 0) : st0;
                const uint32_t end_bit = k < nbnd ? (uint32_t)S.bpos[k] * 8u : limit_bits;
                const uint32_t blk0 = k ? block_base + rem0 + (k - 1) * g.ri_blocks : block_base;
                const uint32_t want = min(k ? g.ri_blocks : rem0, block_end > blk0 ? block_end - blk0 : 0u);
                wc.block = blk0;
                uint32_t got;
                const uint32_t fin = write_span<false>(S, S.clean, g, start, end_bit, end_bit, &got, &wc);
                // the interval must end on its boundary, between MCUs, with exactly its blocks
                if (got != want || (fin & 511u) != 0 || (fin >> 9) != end_bit) wc.bad = 1;
            }
            bad |= wc.bad;
            {
                // DC values of the blocks whose DC was decoded here (the chunk may begin inside a block)
                const uint32_t dc_lo = block_base + ((st0 & 63u) ? 1u : 0u);
                block_base = min(block_base + rem0 + (n_iv - 1) * g.ri_blocks, block_end);
                dc_prefix(S.dc_val, S.dc_flag, g, coef, coef + side_rel, dc_lo, min(block_base, g.n_blocks), dc_carry);
            }
            st0 = pack_state(0, 0, 0);
            dc_carry[0] = dc_carry[1] = dc_carry[2] = 0;
            if (last) { cs = rhi; break; }
            __syncthreads();
            const int32_t next_cs = (int32_t)S.bcast[2];
            if (next_cs <= cs || next_cs > rhi) { bad = 1; cs = rhi; break; }
            cs = next_cs;
            marker_base += nbnd;  // the next chunk starts just after the last marker of this one
            continue;
        }

        // ---- long intervals: speculative subsequences ------------------------------------
        // a chunk that is not the last keeps a tail back so that no symbol straddles its end
        const uint32_t own_bits = last ? limit_bits
                                       : (clean_len > (uint32_t)kChunkTail ? (clean_len - kChunkTail) * 8u : 0u);
        // What a lane takes: a subsequence, or, in the hypothesis passes of the smallest calls,
        // half of one (the passes are shorter, and a chunk of a small window has the lanes for
        // twice the rows); a lane's reads stay inside its subsequence's row either way.
        const uint32_t span_bits = kHyp && by_hypotheses && own_bits <= (uint32_t)kT * hyp_span_bits ? hyp_span_bits : kSubBits;
        const uint32_t nsub = (own_bits + span_bits - 1) / span_bits;  // <= kT
        const bool active = (uint32_t)tid < nsub;
        const uint32_t end_bit = min(((uint32_t)tid + 1u) * span_bits, own_bits);

        uint32_t in_state = tid == 0 ? st0 : pack_state((uint32_t)tid * span_bits, 0, 0);
        uint32_t out_state = in_state, nblk = 0;
        if (by_hypotheses) {
            // ---- the true states by place-in-MCU hypotheses ------------------------------
            // Subsequences [0, first) are settled; x = true state where subsequence `first`
            // begins.  A region is the next kT / H subsequences (H = blocks per MCU), lane
            // tid = j H + h working on subsequence first + j (row j) under hypothesis h.
            //   pass 0: decode from (first bit of the subsequence, block h of an MCU, DC), no
            //           matter where a symbol really begins there; the lanes of row 0 know the
            //           true state and decode from it.  End states -> cand[].
            //   pass 1: decode again from cand[] of the row before: these are the candidates
            //           for the true state at the row's start.  End states -> next[].
            //   link[] of a lane: which candidate of its own row its end state next[] equals.
            //   Lane 0 then follows the links from row to row.  Where the true state is none
            //   of the candidates (the true decoder had not fallen into step with any
            //   hypothesis by the end of the row before), the lanes of that row decode it
            //   once more from the true state, as row 0 did, and the walk goes on from there.
            __shared__ uint16_t hyp_blocks[kT];
            __shared__ uint8_t link[kT], chosen[kT];
            uint32_t *cand = reinterpret_cast<uint32_t *>(S.bpos);  // (the list of interval starts
            uint32_t *next = cand + kT;                             // is of no use to these passes)
            static_assert(sizeof(S.bpos) >= 2 * kT * sizeof(uint32_t), "cand[] and next[] fit");
            // (With 2 KB more only two workgroups fitted, which the compiler's occupancy of three does not tell:
            // calls of gray images that make more than 512 of them took 133 us instead of 89.)
            static_assert(workgroups_by_lds(sizeof(S) + sizeof(hyp_blocks) + sizeof(link) + sizeof(chosen)) >= 3 || !kHyp,
                          "three workgroups a compute unit, as the launch bounds say");
            constexpr uint32_t kNoLink = 255;
            const uint32_t H = g.bpm, per = (uint32_t)kT / H;
            const uint32_t j = (uint32_t)tid / H, h = (uint32_t)tid - j * H;
            uint32_t first = 0, x = st0;
            for (uint32_t region = 0; region < nsub && first < nsub; region++) {
                const uint32_t cnt = min(per, nsub - first);
                const bool mine = j < cnt;
                const uint32_t s_end = min((first + j + 1u) * span_bits, own_bits);
                // which candidate of my row my end state equals (rows link to themselves: the
                // state where row j + 1 begins is looked up among the ends of row j)
                auto find_link = [&]() {
                    uint32_t hit = kNoLink;
                    for (uint32_t k = 0; k < H; k++)
                        if (cand[j * H + k] == next[tid]) { hit = k; break; }
                    link[tid] = (uint8_t)hit;
                };
                for (int pass = 0; pass < 2; pass++) {
                    const bool run = mine && (pass == 0 || j != 0);
                    if (run) {
                        const uint32_t from = pass == 0 ? (j == 0 ? x : pack_state((first + j) * span_bits, h, 0))
                                                        : cand[(uint32_t)tid - H];
                        uint32_t to = from, nb = 0;
                        // (a state past the subsequence's end: the lane before ran through it)
                        if ((from >> 9) < s_end) to = count_span<true>(S, S.clean + clean_row_of_bit(from >> 9), runs, g, from, s_end, limit_bits, &nb);
                        if (pass == 0) cand[tid] = to;
                        if (pass == 1 || j == 0) { next[tid] = to; hyp_blocks[tid] = (uint16_t)nb; }
                    }
                    __syncthreads();
                }
                // (row 0's own candidates are all the true end state: it links to candidate 0)
                if (mine) find_link();
                if (tid == 0) S.bcast[5] = 0;
                __syncthreads();
                // rows [0, walked) are settled; chosen[r] = the lane of row r that decoded from
                // the true state
                for (uint32_t walk = 0; walk < cnt; walk++) {
                    if (tid == 0) {
                        uint32_t r = S.bcast[5], k = 0;  // row r holds the true state in every lane
                        chosen[r] = 0;
                        for (r++; r < cnt; r++) {
                            k = link[(r - 1u) * H + k];
                            if (k == kNoLink) break;
                            chosen[r] = (uint8_t)k;
                        }
                        S.bcast[5] = r;
                    }
                    __syncthreads();
                    const uint32_t r = S.bcast[5];
                    if (r >= cnt) break;
                    // row r begins in a state that is no candidate: decode it from that state
                    if (j == r) {
                        const uint32_t from = next[(r - 1u) * H + chosen[r - 1u]];
                        uint32_t to = from, nb = 0;
                        if ((from >> 9) < s_end) to = count_span<true>(S, S.clean + clean_row_of_bit(from >> 9), runs, g, from, s_end, limit_bits, &nb);
                        next[tid] = to;
                        hyp_blocks[tid] = (uint16_t)nb;
                    }
                    __syncthreads();
                    if (j == r) find_link();
                    __syncthreads();
                }
                if ((uint32_t)tid >= first && (uint32_t)tid < first + cnt) {
                    const uint32_t r = (uint32_t)tid - first;
                    in_state = r == 0 ? x : next[(r - 1u) * H + chosen[r - 1u]];
                    out_state = next[r * H + chosen[r]];
                    nblk = hyp_blocks[r * H + chosen[r]];
                    S.state[tid] = out_state;
                }
                x = next[(cnt - 1u) * H + chosen[cnt - 1u]];
                first += cnt;
                __syncthreads();  // cand[], next[] and the rest are free again
            }
            if (!active) S.state[tid] = out_state;
        } else {
        // synchronise: iterate end states to their fixed point.  After the first round few rows
        // have a new start state, but up to a round's end they are all over the workgroup: they
        // are dealt to neighbouring lanes, or three to four waves a round would decode for a few lanes
        // each.  Start states come back, where a row's predecessor is decoded from another state and
        // falls into step all the same: a row's lane keeps its last three results, and rows are
        // decoded only once nothing moves by those.  (64 full-HD images at quality 95: 14.4 rounds
        // a chunk without, 8.2 with three, no fewer with eight; kernel 1358 -> 1001 us with zeros stored first.)
        RowLists &rows = S.rows();
        if (active) out_state = count_span<true>(S, S.clean + clean_row_of_bit(in_state >> 9), runs, g, in_state, end_bit, limit_bits, &nblk);
        S.state[tid] = out_state;
        uint32_t in1 = ~0u, out1 = 0, nblk1 = 0, in2 = ~0u, out2 = 0, nblk2 = 0;
        __syncthreads();
        // (the first row whose start state is not final becomes final with every decode, and rows
        // behind it move by kept results at most once each in between)
        for (uint32_t round = 0; round <= nsub * nsub; round++) {
            const uint32_t prev_state = tid > 0 ? S.state[tid - 1] : st0;
            const bool moved = active && tid > 0 && prev_state != in_state;
            const bool kept = moved && (prev_state == in1 || prev_state == in2), again = moved && !kept;
            const uint64_t ones = __ballot(again);
            if (__ballot(kept) != 0 && (tid & 63) == 0) S.scan_a[tid >> 6] = 0x10000u | (uint32_t)__popcll(ones);
            else if ((tid & 63) == 0) S.scan_a[tid >> 6] = (uint32_t)__popcll(ones);
            __syncthreads();
            uint32_t at = 0, total = 0;
            for (int ww = 0; ww < kT / 64; ww++) {
                if (ww < tid >> 6) at += S.scan_a[ww];
                total += S.scan_a[ww];
            }
            if (total == 0) break;  // (uniform over the workgroup)
            if (moved && (kept || total < 0x10000u)) {
                // the current result becomes the second, an older one the current one
                const bool second = prev_state == in1;
                const uint32_t o = second ? out1 : out2, n = second ? nblk1 : nblk2;
                if (!second) { in2 = in1; out2 = out1; nblk2 = nblk1; }
                in1 = in_state; out1 = out_state; nblk1 = nblk;
                in_state = prev_state; out_state = o; nblk = n;
            }
            if (total >= 0x10000u) {
                if (kept) S.state[tid] = out_state;
                __syncthreads();
                continue;
            }
            if (again) {
                at += (uint32_t)__popcll(ones & ((1ull << (tid & 63)) - 1ull));
                rows.from[at] = in_state;
                rows.row[at] = (uint8_t)tid;
            }
            __syncthreads();
            if ((uint32_t)tid < total) {
                const uint32_t row = rows.row[tid], from = rows.from[tid], row_end = min((row + 1u) * span_bits, own_bits);
                uint32_t o = from, nb = 0;
                // a predecessor that already ran past the subsequence leaves nothing to decode
                if ((from >> 9) < row_end) o = count_span<true>(S, S.clean + clean_row_of_bit(from >> 9), runs, g, from, row_end, limit_bits, &nb);
                S.state[row] = o;
                rows.blocks[row] = (uint16_t)nb;
            }
            __syncthreads();
            if (again) {
                out_state = S.state[tid];
                nblk = rows.blocks[tid];
            }
        }
        }

        // write: decode once more from the true states
        uint32_t total_blocks;
        const uint32_t my_block = block_base + block_excl_scan(active ? nblk : 0u, S.scan_a, &total_blocks);
        wc.block = my_block;
        // a lane that begins on an MCU boundary where an interval ends must meet the boundary
        // first; lane 0 of a chunk may begin just after one (start of the run, or a boundary
        // consumed at the very end of the previous chunk)
        const bool boundary_due = (in_state & 511u) == 0 && g.ri_blocks != 0 && my_block % g.ri_blocks == 0 &&
                                  my_block < g.n_blocks && tid != 0;
        wc.iv_rem = boundary_due ? 0 : g.ri_blocks ? (int32_t)(g.ri_blocks - my_block % g.ri_blocks) : 0x7FFFFFFF;
        uint32_t final_state = out_state;
        if (active && (in_state >> 9) < end_bit) {
            uint32_t nb2;
            final_state = write_span<true>(S, S.clean + clean_row_of_bit(in_state >> 9), g, in_state, end_bit, limit_bits, &nb2, &wc);
            if (final_state != out_state || nb2 != nblk) wc.bad = 1;
        }
        bad |= wc.bad;
        __syncthreads();
        if (tid == 0) S.bcast[0] = nsub ? S.state[nsub - 1] : st0;
        __syncthreads();
        const uint32_t fs = S.bcast[0];  // true end state of the chunk
        {
            // DC values of the blocks whose DC was decoded in this chunk: it may begin inside
            // a block (DC decoded earlier) and end inside one (DC decoded here)
            const uint32_t dc_lo = block_base + ((st0 & 63u) ? 1u : 0u);
            const uint32_t dc_hi = block_base + total_blocks + ((fs & 63u) ? 1u : 0u);
            dc_prefix(S.dc_val, S.dc_flag, g, coef, coef + side_rel, dc_lo, min(dc_hi, g.n_blocks), dc_carry);
        }

        // carry the true end state into the next chunk
        block_base += total_blocks;
        if (last) { cs = rhi; st0 = fs; break; }
        // raw position of the clean byte the end state points into
        const uint32_t pbit = fs >> 9;
        const uint32_t qc = pbit >> 3;
        if (qc >= clean_len || nsub == 0) {
            // cannot happen for a chunk that is not the last; stop rather than loop
            bad = 1;
            cs = rhi;
            break;
        }
        if (tid == 0) S.bcast[1] = S.bcast[3] = 0;
        __syncthreads();
        {
            // restart markers of this chunk that the next chunk will not stage again: those whose
            // interval begins at or before the clean byte the next chunk starts with
            const unsigned long long m = ((unsigned long long)S.bmask[2 * tid + 1] << 32) | S.bmask[2 * tid];
            const uint32_t first = (uint32_t)tid * 64u;
            if (m != 0 && qc >= first)
                atomicAdd(&S.bcast[3], qc - first >= 63u ? (uint32_t)__popcll(m)
                                                         : (uint32_t)__popcll(m & ((2ull << (qc - first)) - 1ull)));
        }
        if constexpr (!kHyp) keep = S.keep[tid];
        if (S.keep_off[tid] <= qc && qc < S.keep_off[tid] + (uint32_t)__popcll(keep)) {
            unsigned long long m = keep;
            const uint32_t skip = qc - S.keep_off[tid];
            for (uint32_t i = 0; i < skip; i++) m &= m - 1;  // drop the lowest set bits
            S.bcast[1] = (uint32_t)(my_lo + (int32_t)__builtin_ctzll(m));
        }
        __syncthreads();
        const int32_t next_cs = (int32_t)S.bcast[1];
        if (next_cs <= cs || next_cs >= rhi) { bad = 1; cs = rhi; break; }  // no progress: refuse to spin
        cs = next_cs;
        st0 = pack_state(pbit & 7u, (fs >> 6) & 7u, fs & 63u);
        marker_base += S.bcast[3];
    }

    // the run must end on an MCU boundary with exactly the blocks it should hold
    if (tid == 0 && (block_base != block_end || (st0 & 511u) != 0)) bad = 1;
    if (__syncthreads_or(bad)) {
        if (tid == 0) atomicMin(&status[img], (int32_t)PREP_E_CORRUPT);
    }
}

// ---- streams without restart markers ------------------------------------------------
//
// decode_entropy gives such a stream to one workgroup, which walks it chunk by chunk and, in
// every chunk, iterates until the states at the subsequence borders settle: a chain as long as
// the file (a full-HD still: 14 ms) on a chip that is idle otherwise.  Here the stream is cut
// into windows, one workgroup each, that are decoded side by side without knowing the state in
// which the stream enters them.  What takes long to fall into step is the block's place in the
// MCU; bit position and zig-zag index do so within a block or two.  So:
//
//   resolve_streams  A window's clean bytes are cut into rows of row_bytes; lane (j, h) decodes
//       row j from its first bit with the hypothesis "block h of an MCU begins here" (pass 0) and
//       then row j + 1 from the state it reached (pass 1): a node.  A node's end state is looked
//       up among the pass-0 ends of its own row: the equal one is where a node of the next row
//       begins.  An end state that is none of them (1 to 10 % of the nodes, in dense streams most)
//       gets an extra node in the next row, one for all that end in it, decoded in a further
//       pass with the others of its kind.  (There are 128 places.  A window of a 4:2:0 stream of 23
//       bytes per block took 200 to 320 with one for each node, of 19 bytes 36 to 76 shared.)  The last
//       rows, the overlap, are the first rows of the next window: where a chain of nodes meets
//       one of the hypotheses there, the next window has the node that goes on from it.  So every
//       entry (overlap row, hypothesis) leads to an exit of the same form and a count of blocks.
//   chain_streams    follows the entries from window to window of an image: the true chain.
//   write_streams    decodes every window's rows once more, from the true states.
//   finish_window    DC differences -> DC values (in decode_entropy's launch).
//
// Whatever does not fit this scheme (a chain that meets no hypothesis within the overlap, markers
// inside the data, a stream that ends in the wrong state) is set in retry[], and decode_entropy
// decodes the image, and judges it, as if there were no windows.
//
// The work is 2 H + 1 decodes of every byte (H = blocks per MCU) against about ten by iteration
// over 4:2:0, but none waits for another for longer than a row.  Whole calls, one workgroup per
// image against windows: a 44 KB photograph 1099 -> 93 us, a 760 KB full-HD still 14 639 -> 124 us,
// 128 photographs (5 MB) 1879 -> 371 us, 512 thumbnails of 4:4:4, 4:2:0 and gray (5.6 MB)
// 1062 -> 369 us.  Where windows do not pay, api.cpp does not cut (StreamCut).  resolve_streams and
// write_streams are bound by a lane's dependent symbols (about 0.1 us each when the chip is idle) and,
// a third of their time where it is full, by waiting for a window's records, tables and bytes:
// 114 and 79 us of the 128 photographs' 371.

namespace {

constexpr uint32_t kToEnd = 254, kNoWay = 255;       // instead of an exit or an entry
constexpr uint32_t kExit = 0x8000, kNodeToEnd = 0xFFFE, kNodeNoWay = 0xFFFF;  // instead of a next node
// Extra nodes are kept by the state they begin in and their row, in a table with open addressing.
constexpr uint32_t kStateBits = 25, kNoKey = 0xFFFFFFFFu;
constexpr int kExtraProbes = kStreamExtras;          // places looked at; a node without one has no way on
constexpr uint32_t kOpenLimit = 1u << 22;            // bit limit of a window that the data go on after
constexpr int kStreamSlack = 32;                     // raw bytes staged behind the overlap
// clean words of a window: its own bytes and, where every byte is stuffed, the overlap's at half
// their raw number, or twice as many where none is; then zeros
constexpr int kStreamWords = (int)(stream_window_bytes(3, kStreamRowBytes) + 2 * stream_overlap(kStreamRowBytes) * kStreamRowBytes +
                                   kStreamSlack + 64) / 4;
static_assert(stream_rows(1) <= stream_rows(3) && stream_rows(4) <= stream_rows(3) && stream_rows(6) <= stream_rows(3),
              "4:4:4 has the largest windows");

static_assert(kStreamWords * 32 < (1 << (kStateBits - 9)) && kStreamMaxRows < (1 << (32 - kStateBits)) && kStreamExtras == 128,
              "a state and its row fit a key, and the table's size wraps by a mask");

template <typename Tables>
struct StreamShared {
    uint32_t clean[kStreamWords];    // the window's bytes without stuffing, big-endian packed
    Tables tab;
    uint32_t scan_a[kT / 64 + 1];
    uint32_t bcast[4];
};

struct StreamPart {                  // what staging found
    uint32_t own, total;             // clean bytes of the window itself, and with what follows
    bool to_end;                     // the staged bytes reach the end of the data
    bool marker;                     // a marker other than stuffing lies among them, or too little
                                     // is left between long runs of fill bytes
};

// The raw bytes [w * step, (w + 1) * step) of the segment and enough after them for the overlap rows,
// on their way into registers: 16-byte aligned parts that cover them, one or two to a lane, with
// the byte before each part (the segment's first byte has none) and the one after it.  They
// are asked for as long as the host found the segment to be, before anything is known of where the
// data end in it.  (A workgroup that waits for its tables, its window's record and these one after
// the other spends a third of its time waiting where all are asked for together.)
struct StreamLoads {
    int32_t cs, my_lo, per;
    uint4 v[2];
    uint32_t prev[2], after[2];
    __device__ inline StreamLoads(const uint8_t *seg, uint32_t entropy_len, uint32_t w, uint32_t step, uint32_t row_bytes)
    {
        cs = (int32_t)(w * step);
        const int32_t ce = (int32_t)min(w * step + step + 2u * stream_overlap(row_bytes) * row_bytes + kStreamSlack, entropy_len);
        const int32_t a0 = cs - (int32_t)((uintptr_t)(seg + cs) & 15u);
        per = (ce - a0 + 15) >> 4 > kT ? 2 : 1;
        static_assert(kStreamWords * 4 <= 2 * kT * 16, "two parts a lane hold a window");
        my_lo = a0 + (int32_t)threadIdx.x * per * 16;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int32_t plo = my_lo + 16 * k;
            v[k] = make_uint4(0, 0, 0, 0);
            prev[k] = after[k] = 0;
            if (k < per && plo < ce) {
                v[k] = *reinterpret_cast<const uint4 *>(seg + plo);
                if (plo > 0) prev[k] = load_byte(seg + plo - 1);
                if (plo + 16 < (int32_t)entropy_len) after[k] = load_byte(seg + plo + 16);
            }
        }
    }
};

// Stage them in S.clean.  All lanes must call.
template <typename Tables>
__device__ inline StreamPart stage_stream(StreamShared<Tables> &S, const StreamLoads &loads, uint32_t data_len, uint32_t step,
                                          uint32_t row_bytes)
{
    const int tid = threadIdx.x;
    const int32_t cs = loads.cs, own_end = (int32_t)min((uint32_t)cs + step, data_len);
    const int32_t ce = (int32_t)min((uint32_t)cs + step + 2u * stream_overlap(row_bytes) * row_bytes + kStreamSlack, data_len);
    StreamPart part;
    part.to_end = ce == (int32_t)data_len;
    uint32_t keep[2] = {0, 0}, bound = 0;
    int32_t bad = 0;
    uint32_t n_own = 0, n_all = 0;
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int32_t plo = loads.my_lo + 16 * k;
        if (k < loads.per && plo < ce) {
            // (after the data's last byte comes the FF of the marker there)
            const uint32_t after = plo + 16 < (int32_t)data_len ? loads.after[k] : 0xFFu;
            uint32_t b = 0, last;
            classify16(loads.v[k], loads.prev[k], after, plo, cs, ce, &keep[k], &b, &last, &bad);
            bound |= b;
            const int32_t left = own_end - plo;
            const uint32_t mine = left >= 16 ? 0xFFFFu : left > 0 ? (1u << left) - 1u : 0u;
            n_own += (uint32_t)__popcll(keep[k] & mine);
            n_all += (uint32_t)__popcll(keep[k]);
        }
    }
    uint32_t totals;
    const uint32_t before = block_excl_scan(n_all | (n_own << 16), S.scan_a, &totals) & 0xFFFFu;
    part.total = totals & 0xFFFFu;
    part.own = totals >> 16;
    // zeros behind the data: its last word is put together with OR, and lookups near the end
    // read a few words past it
    if (tid < 6) S.clean[(part.total >> 2) + (uint32_t)tid] = 0;
    part.marker = __syncthreads_or(bound != 0 || bad != 0) != 0;
    BytePacker pack(before);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        if (keep[k] == 0) continue;
        const uint32_t wv[4] = {loads.v[k].x, loads.v[k].y, loads.v[k].z, loads.v[k].w};
#pragma unroll
        for (int e = 0; e < 4; e++)
            pack.add(wv[e], (keep[k] >> (4 * e)) & 15u, [&](uint32_t at, uint32_t word) { S.clean[at] = word; });
    }
    __syncthreads();
    if (pack.n != 0) atomicOr(&S.clean[pack.word], pack.rest());
    // Windows are joined at rows that both hold whole, with the bytes of a symbol that begins at
    // their end.  Stuffing leaves at least half of the bytes, which is enough (see ce), but a
    // run of fill bytes (FF FF .. FF 00) may leave any number, behind this window or in it.
    const uint32_t shared = stream_overlap(row_bytes) * row_bytes;
    if ((!part.to_end && part.total - part.own < shared + 8u) || (own_end < (int32_t)data_len && part.own < shared))
        part.marker = true;
    __syncthreads();
    return part;
}

// The rows of a window: row j < n_own holds clean bytes of the window itself, the rows after them
// are the first of the next window.
struct StreamRows {
    uint32_t row_bytes, own, total, n_own, n, limit_bits;
    bool to_end;  // the data end with the last row
    __device__ inline StreamRows(const StreamPart &p, uint32_t rb) : row_bytes(rb), own(p.own), total(p.total)
    {
        n_own = (own + rb - 1) / rb;
        n = n_own + min((total - own + rb - 1) / rb, stream_overlap(rb));
        to_end = p.to_end && total - own <= stream_overlap(rb) * rb;
        limit_bits = p.to_end ? total * 8u : kOpenLimit;
    }
    __device__ inline uint32_t start(uint32_t j) const { return 8u * (j < n_own ? j * row_bytes : own + (j - n_own) * row_bytes); }
    __device__ inline uint32_t end(uint32_t j) const { return 8u * (j < n_own ? min((j + 1u) * row_bytes, own) : min(own + (j - n_own + 1u) * row_bytes, total)); }
};

// The extra node of key (see kStateBits), made if there is none yet; x = where to look first.  Out of
// line: inlined, it cost resolve_streams 3 % in calls that need few.
__device__ __attribute__((noinline)) uint32_t extra_node(uint32_t *keys, uint32_t *n_extra, uint32_t key, uint32_t x)
{
    for (int probe = 0; probe < kExtraProbes; probe++, x = (x + 1u) & (uint32_t)(kStreamExtras - 1)) {
        const uint32_t was = atomicCAS(&keys[x], kNoKey, key);
        if (was == kNoKey) atomicAdd(n_extra, 1u);
        if (was == kNoKey || was == key) return (uint32_t)kT + x;
    }
    return kNodeNoWay;
}

}  // namespace

__global__ __launch_bounds__(kDecodeThreads) void resolve_streams(
    const uint8_t *__restrict__ bits, const ImageRec *__restrict__ recs, int n_images, uint32_t row_bytes,
    const uint32_t *__restrict__ data_end, uint32_t *__restrict__ retry, const uint4 *__restrict__ tables,
    StreamWindow *__restrict__ windows)
{
    __shared__ StreamShared<HuffTables> S;
    __shared__ uint32_t cand[kT];              // end states of pass 0
    __shared__ uint32_t node_end[kStreamNodes];
    __shared__ uint16_t node_blocks[kStreamNodes], node_next[kStreamNodes];
    __shared__ uint32_t extra_key[kStreamExtras];  // extra nodes: row << 25 | state in which it begins, or kNoKey
    __shared__ uint32_t n_extra;
    const int tid = threadIdx.x;
    const uint32_t wg = blockIdx.x;
    const int img = image_of_stream(recs, n_images, wg);
    const ImageRec &R = recs[img];
    const uint32_t w = wg - R.stream0;
    if (w >= R.n_streams) return;
    Geometry g;
    stream_geometry(g, R);
    const uint32_t H = g.bpm, step = stream_window_bytes(H, row_bytes);
    const StreamLoads loads(bits + R.file_off + R.entropy_rel, R.entropy_len, w, step, row_bytes);
    const uint32_t data_len = min(R.entropy_len, data_end[img]);
    StreamWindow &W = windows[wg];
    if (w * step >= data_len) {
        // the data ended before this window; an empty segment is decode_entropy's to judge
        if (tid == 0 && w == 0) retry[img] = 1;
        if (tid < kStreamEntries) W.through[tid] = kNoWay;
        return;
    }
    load_tables(S.tab, tables, R.table_slot);
    if (tid < kStreamExtras) {
        extra_key[tid] = kNoKey;
        node_next[kT + tid] = kNodeNoWay;
        node_blocks[kT + tid] = 0;
    }
    if (tid == 0) n_extra = 0;
    const StreamPart part = stage_stream(S, loads, data_len, step, row_bytes);
    if (part.marker && tid == 0) retry[img] = 1;
    const StreamRows rows(part, row_bytes);

    const uint32_t j = (uint32_t)tid / H, h = (uint32_t)tid - j * H;
    const bool mine = j < rows.n && j < stream_rows(H);
    uint32_t state = 0, nb = 0;
    if (mine) {
        state = count_span<false>(S, S.clean, S.tab.run, g, pack_state(rows.start(j), h, 0), rows.end(j), rows.limit_bits, &nb);
        cand[tid] = state;
    }
    __syncthreads();
    // where node id, whose row r ends in state s, goes on
    auto link = [&](uint32_t id, uint32_t r, uint32_t s) {
        uint32_t k = 0;
        while (k < H && cand[r * H + k] != s) k++;
        uint32_t to = kNodeNoWay;
        if (k < H && r >= rows.n_own) {
            to = kExit | ((r - rows.n_own) * H + k);  // in an overlap row: the next window goes on from there
        } else if (r + 1u >= rows.n) {
            if (rows.to_end) to = kNodeToEnd;
        } else if (k < H) {
            to = (r + 1u) * H + k;
        } else {
            // (nodes that begin alike are one: all decoders that are in step come here in the same
            // state where no hypothesis of the row has fallen into step by its end)
            to = extra_node(extra_key, &n_extra, ((r + 1u) << kStateBits) | s, (s * 0x9E3779B1u) >> 26);
        }
        node_next[id] = (uint16_t)to;
    };
    // pass 1 (row 0 begins in a known state in window 0, and is not entered otherwise; an overlap
    // row after the first is entered by extra nodes only)
    const bool node = mine && j <= rows.n_own;
    if (node) {
        if (j != 0) {
            const uint32_t from = cand[(uint32_t)tid - H];
            state = from;
            nb = 0;
            // (a state past the row's end: the row before ran through it)
            if ((from >> 9) < rows.end(j)) state = count_span<false>(S, S.clean, S.tab.run, g, from, rows.end(j), rows.limit_bits, &nb);
        }
        node_end[tid] = state;
        node_blocks[tid] = (uint16_t)nb;
        if (j == 0) node_next[tid] = (uint16_t)(rows.n > 1 ? (uint32_t)tid + H : rows.to_end ? kNodeToEnd : kNodeNoWay);
        else link((uint32_t)tid, j, state);
    } else {
        node_next[tid] = kNodeNoWay;
        node_blocks[tid] = 0;
        node_end[tid] = 0;
    }
    __syncthreads();
    // the extra nodes, a lane each, a generation at a time (a generation's are at least one row further)
    static_assert(kStreamExtras <= kT, "a lane per extra node");
    bool mine_done = false;
    uint32_t done = 0;
    for (uint32_t round = 0; round < (uint32_t)kStreamMaxRows; round++) {
        const uint32_t have = n_extra, key = tid < kStreamExtras ? extra_key[tid] : kNoKey;
        __syncthreads();
        if (done == have) break;
        if (key != kNoKey && !mine_done) {
            const uint32_t from = key & ((1u << kStateBits) - 1u), r = key >> kStateBits;
            uint32_t to = from, n = 0;
            if ((from >> 9) < rows.end(r)) to = count_span<false>(S, S.clean, S.tab.run, g, from, rows.end(r), rows.limit_bits, &n);
            node_end[kT + tid] = to;
            node_blocks[kT + tid] = (uint16_t)n;
            link((uint32_t)(kT + tid), r, to);
            mine_done = true;
        }
        done = have;
        __syncthreads();
    }
    static_assert(kStreamNodes <= 2 * kT, "a lane has two nodes");
    const uint32_t other = (uint32_t)(kT + tid);  // this lane's extra node, if tid < kStreamExtras
    W.end[tid] = node_end[tid];
    W.blocks[tid] = node_blocks[tid];
    W.next[tid] = node_next[tid];
    if (tid < kStreamExtras && extra_key[tid] != kNoKey) {
        W.end[other] = node_end[other];
        W.blocks[other] = node_blocks[other];
        W.next[other] = node_next[other];
    }
    // From every node to the end of its chain, by twice as many nodes a round (a chain has at most one
    // node per row): node_next leads there, node_end becomes the blocks on the way.  (One lane an entry, node
    // by node, took 5 of the 27 us of a call with one photograph.)
    node_end[tid] = node_blocks[tid];
    if (tid < kStreamExtras) node_end[other] = node_blocks[other];
    for (uint32_t reach = 1; reach < rows.n; reach *= 2) {
        __syncthreads();
        uint32_t next[2] = {kNodeNoWay, kNodeNoWay}, more[2] = {0, 0};
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (k == 1 && tid >= kStreamExtras) continue;
            next[k] = node_next[tid + k * kT];
            if (next[k] < (uint32_t)kStreamNodes) {
                more[k] = node_end[next[k]];
                next[k] = node_next[next[k]];
            }
        }
        __syncthreads();
        node_next[tid] = (uint16_t)next[0];
        node_end[tid] += more[0];
        if (tid < kStreamExtras) {
            node_next[other] = (uint16_t)next[1];
            node_end[other] += more[1];
        }
    }
    __syncthreads();
    if (tid < kStreamEntries) {
        // entry e = (overlap row i, hypothesis k) goes on with node (i + 1, k) here; window 0 is
        // entered by node 0
        const uint32_t e = (uint32_t)tid;
        const uint32_t at = w == 0 ? 0u : e + H;
        uint32_t way = kNoWay, blocks = 0;
        if (e < (w == 0 ? 1u : stream_overlap(row_bytes) * H)) {
            W.entry_state[e] = w == 0 ? 0u : cand[e];
            if (w != 0 && e / H + 1u >= rows.n) {
                way = rows.to_end ? kToEnd : kNoWay;  // no such row: all was decoded in the window before
            } else {
                const uint32_t to = node_next[at];
                blocks = node_end[at];
                way = to == kNodeToEnd ? kToEnd : to != kNodeNoWay && (to & kExit) != 0 ? to & ~kExit : kNoWay;
            }
        }
        W.through[e] = (blocks << 8) | way;
    }
}

// One workgroup per image: which entry of each window the image's true chain takes, and the block
// there.  Windows are taken kChainTile at a time; within a tile, lane (s, e) follows segment s from
// entry e, one lane strings the segments together, and a lane per segment goes over it again: as many
// segments as a segment has windows, so that no stage is much longer than the others.  Bound by the
// latency of these walks and of the tile's loads (24 entries a window, in calls with little data 42), which
// are under way together: a full-HD still of 600 windows 32 -> 20 us with sixteen waves instead of four and
// one tile; one of 795 windows 28.6 with a tile of 640, 24.3 with one for all.
constexpr int kChainThreads = 1024;
constexpr int kChainTile = 256;  // windows: 43 KB of LDS
// the larger: all windows that an image can have in a call with short rows (833 of six blocks per MCU: 140 KB)
constexpr int kChainLargeTile = (int)(kStreamTinyBytes / stream_window_bytes(6, kStreamTinyRowBytes)) + 1;
template <int kTile>
__global__ __launch_bounds__(kChainThreads) void chain_streams(
    const ImageRec *__restrict__ recs, uint32_t row_bytes, uint32_t *__restrict__ retry, StreamWindow *__restrict__ windows)
{
    constexpr int kChainLoads = (kTile * kStreamEntries + kChainThreads - 1) / kChainThreads;
    __shared__ uint32_t through[kTile * kStreamEntries];
    __shared__ uint32_t seg_way[kChainThreads], seg_blocks[kChainThreads];
    __shared__ uint32_t seg_entry[kChainThreads], seg_block[kChainThreads];
    __shared__ uint32_t s_entry, s_block;
    static_assert(workgroups_by_lds(sizeof(through) + 4 * sizeof(seg_way) + 8) >= 1, "a tile fits");
    const ImageRec &R = recs[blockIdx.x];
    const int tid = threadIdx.x;
    const uint32_t n = R.n_streams;
    if (n == 0 || R.status != PREP_OK) return;
    const bool redo = retry[blockIdx.x] != 0;
    StreamWindow *W = windows + R.stream0;
    const uint32_t E = stream_overlap(row_bytes) * R.blocks_per_mcu;
    if (tid == 0) {
        s_entry = redo ? kNoWay : 0u;
        s_block = 0;
    }
    for (uint32_t w0 = 0; w0 < n; w0 += kTile) {
        const uint32_t cnt = min(n - w0, (uint32_t)kTile);
        uint32_t v[kChainLoads];
#pragma unroll
        for (int k = 0; k < kChainLoads; k++) {
            const uint32_t i = min((uint32_t)(tid + k * kChainThreads), cnt * E - 1u);
            if ((uint32_t)(k * kChainThreads) < cnt * E) v[k] = W[w0 + i / E].through[i % E];
        }
#pragma unroll
        for (int k = 0; k < kChainLoads; k++)
            if ((uint32_t)(tid + k * kChainThreads) < cnt * E) through[tid + k * kChainThreads] = v[k];
        uint32_t n_seg = 1;
        while (n_seg * n_seg < cnt && (n_seg + 1u) * E <= (uint32_t)kChainThreads) n_seg++;
        __syncthreads();
        const uint32_t len = (cnt + n_seg - 1) / n_seg;
        const uint32_t s = (uint32_t)tid / E, e = (uint32_t)tid - s * E;
        const uint32_t lo = min(s * len, cnt), hi = min(lo + len, cnt);
        if (s < n_seg) {
            uint32_t way = e, blocks = 0;
            for (uint32_t i = lo; i < hi && way < E; i++) {
                const uint32_t t = through[i * E + way];
                blocks += t >> 8;
                way = t & 255u;
            }
            seg_way[tid] = way;
            seg_blocks[tid] = blocks;
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t way = s_entry, block = s_block;
            for (uint32_t i = 0; i < n_seg; i++) {
                seg_entry[i] = way;
                seg_block[i] = block;
                if (way < E) {
                    block += seg_blocks[i * E + way];
                    way = seg_way[i * E + way];
                }
            }
            s_entry = way;
            s_block = block;
        }
        __syncthreads();
        if (e == 0 && s < n_seg) {
            uint32_t way = seg_entry[s], block = seg_block[s];
            for (uint32_t i = lo; i < hi; i++) {
                W[w0 + i].entry = way;
                W[w0 + i].block = block;
                if (way < E) {
                    const uint32_t t = through[i * E + way];
                    block += t >> 8;
                    way = t & 255u;
                }
            }
        }
        __syncthreads();
    }
    // the chain has to reach the end of the data with all of the image's blocks
    // (all lanes have come here past the last barrier: they see the same)
    if (s_entry != kToEnd || s_block != R.n_blocks) {
        for (uint32_t i = (uint32_t)tid; i < n; i += kChainThreads) W[i].entry = kNoWay;
        if (tid == 0) retry[blockIdx.x] = 1;
    }
}

__global__ __launch_bounds__(kDecodeThreads) void write_streams(
    const uint8_t *__restrict__ bits, const ImageRec *__restrict__ recs, int n_images, uint32_t row_bytes,
    const uint32_t *__restrict__ data_end, uint32_t *__restrict__ retry, const uint4 *__restrict__ tables,
    StreamWindow *__restrict__ windows, int16_t *__restrict__ coef_all, uint32_t side_off)
{
    __shared__ StreamShared<HuffCodes> S;
    __shared__ uint32_t node_end[kStreamNodes];
    __shared__ uint16_t node_blocks[kStreamNodes], node_next[kStreamNodes];
    __shared__ uint16_t chain[kStreamMaxRows + 1];
    const int tid = threadIdx.x;
    const uint32_t wg = blockIdx.x;
    const int img = image_of_stream(recs, n_images, wg);
    const ImageRec &R = recs[img];
    const uint32_t w = wg - R.stream0;
    if (w >= R.n_streams || R.status != PREP_OK) return;
    StreamWindow &W = windows[wg];
    const uint32_t H = R.blocks_per_mcu, entry = W.entry, block0 = W.block;
    const uint32_t step = stream_window_bytes(H, row_bytes);
    const StreamLoads loads(bits + R.file_off + R.entropy_rel, R.entropy_len, w, step, row_bytes);
    uint32_t end[2], blocks[2], next[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int i = min(tid + k * kT, kStreamNodes - 1);
        end[k] = W.end[i];
        blocks[k] = W.blocks[i];
        next[k] = W.next[i];
    }
    // An image that is to be decoded in one piece is left alone.  Other windows of it may find that
    // out only now and set retry[img]: that is for the next kernels to read.  Here the waves of this
    // workgroup would read it at different times, and some would leave where others go on to
    // the barriers; what chain_streams wrote is the same for all of them.
    if (entry >= stream_overlap(row_bytes) * H) {
        if (tid == 0) {
            W.dc_lo = W.dc_hi = 0;
            W.dc_sum[0] = W.dc_sum[1] = W.dc_sum[2] = 0;
        }
        return;
    }
    Geometry g;
    stream_geometry(g, R);
    const uint32_t entry_state = W.entry_state[entry];
    const uint32_t data_len = min(R.entropy_len, data_end[img]);
    load_tables(S.tab, tables, R.table_slot);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int i = min(tid + k * kT, kStreamNodes - 1);
        node_end[i] = end[k];
        node_blocks[i] = (uint16_t)blocks[k];
        node_next[i] = (uint16_t)next[k];
    }
    const StreamPart part = stage_stream(S, loads, data_len, step, row_bytes);
    const StreamRows rows(part, row_bytes);
    const uint32_t row0 = w == 0 ? 0u : entry / H + 1u;  // first row of the chain
    if (tid == 0) {
        uint32_t cnt = 0, at = w == 0 ? 0u : entry + H;
        while (row0 + cnt < rows.n) {
            chain[cnt++] = (uint16_t)at;
            at = node_next[at];
            if (at >= (uint32_t)kStreamNodes) break;  // an exit, or the end of the data
        }
        S.bcast[0] = cnt;
    }
    __syncthreads();
    const uint32_t cnt = S.bcast[0];
    const bool active = (uint32_t)tid < cnt;
    const uint32_t row = row0 + (uint32_t)tid;
    uint32_t nblk = 0, in_state = 0, out_state = 0;
    if (active) {
        in_state = tid == 0 ? entry_state : node_end[chain[tid - 1]];
        out_state = node_end[chain[tid]];
        nblk = node_blocks[chain[tid]];
    }
    uint32_t total_blocks;
    const uint32_t my_block = block0 + block_excl_scan(nblk, S.scan_a, &total_blocks);
    const uint32_t exit_state = cnt ? node_end[chain[cnt - 1]] : entry_state;
    int16_t *coef = coef_all + (size_t)R.coef_block0 * 64;
    const uint32_t side_rel = side_off + R.coef_block0 - R.coef_block0 * 64u;
    // Zeros over exactly the coefficients that this window decodes: a block that is under way at
    // either end is shared with the workgroup next door, each with its own part of it.
    const uint32_t all = g.n_blocks * 64u;
    const uint32_t z_lo = min(block0 * 64u + (entry_state & 63u), all);
    const uint32_t z_hi = max(z_lo, min((block0 + total_blocks) * 64u + (exit_state & 63u), all));
    {
        const uint32_t a = min((z_lo + 7u) & ~7u, z_hi), b = max(a, z_hi & ~7u);
        if ((uint32_t)tid < a - z_lo) coef[z_lo + (uint32_t)tid] = 0;
        for (uint32_t u = a + 8u * (uint32_t)tid; u < b; u += 8u * kT)
            *reinterpret_cast<uint4 *>(coef + u) = make_uint4(0, 0, 0, 0);
        if ((uint32_t)tid < z_hi - b) coef[b + (uint32_t)tid] = 0;
    }
    __syncthreads();  // (and only then does any lane store a coefficient)
    WriteCtx wc;
    wc.coef = coef;
    wc.side_rel = side_rel;
    wc.block = my_block;
    wc.iv_rem = 0;
    wc.bad = 0;
    if (active) {
        uint32_t fin = in_state, got = 0;
        if ((in_state >> 9) < rows.end(row)) fin = write_span<false>(S, S.clean, g, in_state, rows.end(row), rows.limit_bits, &got, &wc);
        if (fin != out_state || got != nblk) wc.bad = 1;
        // the data end between MCUs
        if (rows.end(row) == rows.limit_bits && ((fin & 511u) != 0 || (fin >> 9) != rows.limit_bits)) wc.bad = 1;
    }
    if (__syncthreads_or(wc.bad) && tid == 0) retry[img] = 1;
    // the DC differences' sums, for the windows after this one
    const uint32_t dc_lo = min(block0 + ((entry_state & 63u) ? 1u : 0u), g.n_blocks);
    const uint32_t dc_hi = max(dc_lo, min(block0 + total_blocks + ((exit_state & 63u) ? 1u : 0u), g.n_blocks));
    uint32_t sum[3] = {0, 0, 0};
    const int16_t *side = coef + side_rel;
    for (uint32_t i = dc_lo + (uint32_t)tid; i < dc_hi; i += kT) {
        const uint32_t c = comp_of_block(g, i % H);
        const uint32_t d = (uint32_t)(int32_t)side[i];
        sum[0] += c == 0 ? d : 0u;
        sum[1] += c == 1 ? d : 0u;
        sum[2] += c == 2 ? d : 0u;
    }
#pragma unroll
    for (int c = 0; c < 3; c++) {
        sum[c] = block_sum(sum[c], S.scan_a);
        if (tid == 0) W.dc_sum[c] = (int32_t)sum[c];
    }
    if (tid == 0) {
        W.dc_lo = dc_lo;
        W.dc_hi = dc_hi;
    }
}

size_t huff_tables_bytes() { return sizeof(HuffTables); }
static_assert(sizeof(HuffTables) % 16 == 0 && sizeof(HuffCodes) % 16 == 0 && sizeof(HuffTables) == sizeof(HuffCodes) + sizeof(HuffTables::run), "table slots are copied in 16-byte units");

void launch_scan_restart_markers(const uint8_t *bits, const ImageRec *recs, int n_images,
                                 uint32_t n_windows, uint32_t window_bytes, uint32_t *win_count, uint32_t *win_first,
                                 uint32_t *data_end, uint32_t *retry,
                                 int32_t *status, const uint32_t *table_rep, uint32_t n_tables,
                                 bool runs, uint8_t *tables, hipStream_t stream)
{
    if (n_windows == 0) return;
    hipLaunchKernelGGL(scan_restart_markers, dim3(n_windows + 4 * kTableParts * n_tables), dim3(kDecodeThreads), 0, stream,
                       bits, recs, n_images, n_windows, window_bytes, win_count, win_first, data_end, retry, status, table_rep,
                       runs, reinterpret_cast<uint4 *>(tables));
}

void launch_decode_entropy(const uint8_t *bits, const ImageRec *recs, int n_images,
                           uint32_t n_windows, const uint32_t *win_count, const uint32_t *win_first,
                           const uint32_t *data_end, const uint32_t *retry, int16_t *coef, uint32_t side_off, int32_t *status,
                           const uint8_t *tables, bool small_windows, uint32_t hyp_span_bits, bool long_intervals,
                           uint32_t n_streams, const StreamWindow *win, hipStream_t stream)
{
    if (n_windows == 0) return;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(n_windows + n_streams), dim3(kDecodeThreads), 0, stream, bits, recs, n_images, win_count,
                           win_first, data_end, retry, coef, side_off, status, reinterpret_cast<const uint4 *>(tables),
                           hyp_span_bits, n_windows, win);
    };
    if (small_windows) launch(decode_entropy<true, true>);
    else if (long_intervals) launch(decode_entropy<false, true>);
    else launch(decode_entropy<false, false>);
}

void launch_decode_streams(const uint8_t *bits, const ImageRec *recs, int n_images, uint32_t n_streams, uint32_t row_bytes,
                           const uint32_t *data_end, uint32_t *retry, StreamWindow *win, int16_t *coef, uint32_t side_off,
                           const uint8_t *tables, hipStream_t stream)
{
    if (n_streams == 0) return;
    const uint4 *tab = reinterpret_cast<const uint4 *>(tables);
    hipLaunchKernelGGL(resolve_streams, dim3(n_streams), dim3(kDecodeThreads), 0, stream, bits, recs, n_images, row_bytes,
                       data_end, retry, tab, win);
    // the larger tile where images have more windows than half the smaller one (600 windows 24 -> 20 us; 128
    // images of 16 windows 4.8 -> 5.1) and a compute unit has no other image to follow
    if (n_images <= 256 && n_streams > (uint32_t)n_images * (kChainTile / 2))
        hipLaunchKernelGGL(chain_streams<kChainLargeTile>, dim3(n_images), dim3(kChainThreads), 0, stream, recs, row_bytes, retry, win);
    else
        hipLaunchKernelGGL(chain_streams<kChainTile>, dim3(n_images), dim3(kChainThreads), 0, stream, recs, row_bytes, retry, win);
    hipLaunchKernelGGL(write_streams, dim3(n_streams), dim3(kDecodeThreads), 0, stream, bits, recs, n_images, row_bytes,
                       data_end, retry, tab, win, coef, side_off);
}

}  // namespace prep
