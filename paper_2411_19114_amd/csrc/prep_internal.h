// Shared between the host code and the HIP kernels of libprep: plain-old-data
// records that travel to the GPU and the launch geometry constants.
#pragma once
#include <stdint.h>

namespace prep {

constexpr uint32_t kComputeUnits = 256;                     // of the device

// ---- entropy decoder geometry -------------------------------------------
// One workgroup owns a contiguous run of restart intervals of one image and
// decodes it chunk by chunk.  A chunk is kChunkRaw raw bytes staged into LDS
// with stuffing and markers removed; in the speculative regime each lane owns
// one subsequence of kSubseqBytes clean bytes.
constexpr int kDecodeThreads = 256;
constexpr int kSubseqBytes = 64;                            // clean bytes per lane
constexpr int kChunkRaw = kDecodeThreads * kSubseqBytes;    // raw bytes staged per chunk
constexpr int kChunkTail = 16;                              // bytes a non-final chunk keeps back
constexpr int kWindowBytes = 12288;                         // raw bytes between workgroup starts
// A call with little entropy-coded data would leave most of the chip idle behind a few lanes
// that walk whole restart intervals one symbol after the other.  Such a call is cut into
// smaller windows (more workgroups, a few restart intervals each) and its workgroups find the
// decoder states inside an interval by phase hypotheses instead (see decode_entropy).
constexpr int kSmallWindowBytes = 2048;
// Entropy-coded bytes of a call up to which it is cut small.  The chip holds 768 workgroups of that variant, 1.5 MB
// of windows.  Decode stage, us, cut small against not, images of 480 x 360: a marker a row, 4:2:0 98 / 142 (0.6 MB),
// 109 / 140 (1.1), 160 / 140 (1.7); 4:2:2 92 / 263 (1.3), 161 / 262 (2.5), 234 / 343 (3.8); gray 79 / 212 (1.5),
// 149 / 230 (3.1); 4:4:4 80 / 95 (0.5), 88 / 94 (0.9), 135 / 95 (1.8).  Where intervals are much shorter than a
// window the line lies lower: a marker every eight MCUs, 4:2:0 99 / 137 (1.1), 152 / 137 (1.7), but 4:2:2 98 / 89 (0.3),
// 4:4:4 102 / 70 (0.5), gray 104 / 51 (0.3): there the cut does not pay at all, and is made all the same.
constexpr uint64_t kSmallCallBytes = 1536 << 10;
// The smallest calls (a single image, a batch of a few dozen small ones) still leave most
// compute units idle with 2 KiB windows: they are cut into windows of about one restart
// interval of a small image, and a lane of the hypothesis passes takes half a subsequence.
// 768 such windows are 384 KB; beyond them the two ways meet (images of 256 x 256, a marker a row, us, these windows
// against 2 KiB: 4:2:0 56 / 79 at 84 KB, 60 / 80 at 335, 98 / 81 at 503; 4:4:4 61 / 81 at 257, 102 / 82 at 513; gray
// 58 / 93 at 307, 96 / 93 at 461).
constexpr int kTinyWindowBytes = 512;
constexpr uint64_t kTinyCallBytes = 448 << 10;
// Mean bytes of a restart interval up to which a lane decodes it whole, in large calls (see decode_entropy)
constexpr int kLongIntervalBytes = 1024;
// Streams without restart markers are cut into windows too, one workgroup each, where that pays
// (StreamCut in api.cpp; the kernels: resolve_streams in entropy.hip).  A window is decoded in rows,
// a lane to a row and hypothesis; its last rows, the overlap, are the first rows of the next window.
constexpr int kStreamRowBytes = 68;                         // clean bytes per row: 17 words, so that rows begin in different LDS banks
constexpr int kStreamTinyRowBytes = 36;                     // the same in calls with little data
// Entropy-coded bytes of such streams in a call up to which rows are short.  Short rows make more
// workgroups, whose lanes have less to do one after the other; once the chip is full, their longer
// overlaps only add work.  Decode stage, short against long rows, us, images of 480 x 360: 4:2:0 74 against 91 (one,
// 35 KB), 91 / 93 (0.6 MB), 97 / 98 (0.8), 108 / 99 (1.1), 137 / 107 (1.7).  Where fewer hypotheses are decoded the two
// meet later: 4:4:4 98 / 109 (1.8), 148 / 132 (3.6); 4:2:2 87 / 97 (1.2), 103 / 101 (1.9); gray 81 / 92 (2.0), 117 / 104
// (3.1).  One full-HD still of 0.76 MB of noise, near the density limit, loses by them: 146 / 114.
constexpr uint64_t kStreamTinyBytes = 1024 << 10;
// Overlap rows.  A decoder that comes out of a window agrees with none of the hypotheses of an
// overlap row with a probability that falls with the row's length: full-HD stills of quality 95,
// the slowest seen, 10 % for rows of 36 bytes and 1 % for rows of 68 (photographs of quality 90:
// 3 and 1 %).  About 250 bytes leave one in 10^7 windows without a way on, if rows were
// independent of one another; counted, the sparsest streams that failed had 20 bytes per block and
// lost one window in 500 (see stream_density_limit).
constexpr int kStreamMaxOverlap = 7;
inline constexpr uint32_t stream_overlap(uint32_t row_bytes) { return row_bytes == (uint32_t)kStreamTinyRowBytes ? 7 : 4; }
constexpr int kStreamMaxRows = 85;                          // rows per window: 256 lanes over the hypotheses, at most this many
// Streams with more bytes per block than this (in tenths; b = blocks per MCU) are not cut.  The
// longer the blocks, the longer a decoder runs before it falls into step with a hypothesis, and
// beyond these densities too many chains come through an overlap without: the image is then
// decoded twice, which costs 2 to 8 % for one image and a quarter for a batch.  Codes made for the
// image (own; an AC table that leaves symbols out) are nearer to its statistics and take longer to
// fall into step than the codes of T.81 Annex K do.  Of 9 700 images of noise and of shapes, qualities
// 90 to 97, each with short and with long rows, all windows were joined: up to the limits in 99.7 % of
// those of 256 x 256, 99 % of 512 x 384 and 93 % of 1600 x 1200 (which decode 100 times faster then), in
// the next two bytes in 94, 85 and 40 %.  Photographs of quality 90 have 6 to 12 bytes, stills of
// quality 95 15 to 18, noise of 8 levels at quality 95 19 (gray 24), with own codes 18 (22).
inline constexpr uint32_t stream_density_limit(uint32_t b, bool own, uint32_t row_bytes)
{
    const bool short_rows = row_bytes == (uint32_t)kStreamTinyRowBytes;
    if (own) return short_rows ? (b == 1 ? 240 : 175) : (b == 1 ? 260 : 210);
    return short_rows ? (b == 1 ? 260 : 230) : (b == 1 ? 280 : 245);
}
constexpr uint32_t kAnnexKAcSymbols = 162;                  // symbols of an AC table that leaves none out
// Streams of one chunk (kChunkRaw) that are many enough to occupy the chip with a workgroup each
// settle there in few rounds, unless an MCU has six blocks; see StreamCut in api.cpp.
inline constexpr uint32_t stream_full_chip(uint32_t b) { return b <= 3 ? 192 : b == 4 ? 384 : 0xFFFFFFFFu; }
constexpr uint32_t kStreamHalfChip = 128;                   // the same for b <= 3 where the call is past kStreamTinyBytes
constexpr uint32_t kStreamFewBytesCall = 256;               // the same for any b where no stream is longer than
constexpr uint64_t kStreamFewBytes = 512;                   // a few subsequences
inline constexpr uint32_t stream_rows(uint32_t blocks_per_mcu)
{
    return kDecodeThreads / blocks_per_mcu < (uint32_t)kStreamMaxRows ? kDecodeThreads / blocks_per_mcu : (uint32_t)kStreamMaxRows;
}
// raw bytes between window starts
inline constexpr uint32_t stream_window_bytes(uint32_t blocks_per_mcu, uint32_t row_bytes)
{
    return (stream_rows(blocks_per_mcu) - stream_overlap(row_bytes)) * row_bytes;
}
// What the kernels of such streams hand on per window: its decoder states (nodes), where each
// entry into the window leads, and what the chain through the image's windows found.
constexpr int kStreamExtras = 128;                          // nodes besides one per lane
constexpr int kStreamNodes = kDecodeThreads + kStreamExtras;
constexpr int kStreamEntries = kStreamMaxOverlap * 6;         // entries into a window, or exits of it
struct StreamWindow {
    uint32_t end[kStreamNodes];        // state where the node's row ends
    uint16_t blocks[kStreamNodes];     // blocks completed in the row
    uint16_t next[kStreamNodes];       // node of the next row that begins in that state, or a code
    uint32_t entry_state[kStreamEntries];  // state at entry e
    uint32_t through[kStreamEntries];  // from entry e: blocks completed << 8 | exit or code
    uint32_t entry;                    // the entry that the image's true chain takes, or a code
    uint32_t block;                    // block of the image that is under way or next there
    uint32_t dc_lo, dc_hi;             // blocks whose DC difference was decoded in this window
    int32_t dc_sum[3];                 // sums of these differences per component
    uint32_t pad_;
};
// Images of a batch mostly share their Huffman tables (encoders write the tables of T.81
// Annex K unless asked to optimise): each distinct set of four tables is expanded once per
// batch into a slot of device memory and copied into LDS by the workgroups that need it.
constexpr uint32_t kMaxTableSlots = 1024;
constexpr uint32_t kNoTableSlot = 0xFFFFFFFFu;             // expand the tables in the workgroup

// ---- reconstruction geometry ----------------------------------------------
// Sampling modes (the PREP_SAMPLING_* values): luma blocks per MCU along x and y (T.81
// A.1.1, chroma is 1 x 1) and blocks per MCU (A.2.3).
inline constexpr int luma_h(int sampling) { return sampling == 1 || sampling == 3 ? 2 : 1; }
inline constexpr int luma_v(int sampling) { return sampling == 1 || sampling == 4 ? 2 : 1; }
inline constexpr int blocks_per_mcu_of(int sampling)
{
    return sampling == 2 ? 1 : luma_h(sampling) * luma_v(sampling) + 2;
}
// One workgroup turns kReconBlocks 8x8 blocks (a run of MCUs of one MCU row)
// into RGB pixels: 5 MCUs of 4:2:0, 10 of 4:4:4, 8 of 4:2:2 or 4:4:0, 32 of grayscale.
constexpr int kReconThreads = 256;
constexpr int kReconBlocks = 32;
inline constexpr int recon_mcus_per_group(int sampling) { return kReconBlocks / blocks_per_mcu_of(sampling); }
// A workgroup takes up to kReconMaxGroupsPerWg consecutive groups of one image: as many as
// leave about kReconGroupsPerWgDivisor workgroups in the launch (two rounds of a full chip).
constexpr uint32_t kReconMaxGroupsPerWg = 8;
constexpr uint32_t kReconGroupsPerWgDivisor = 3072;

// Per-image record, written by the host parser (T.81 Annex B) and read by
// every kernel.  file_off is the byte offset of the file in the device copy of
// the batch's bitstreams; entropy_rel, dht_off and dqt_off count from there.
struct ImageRec {
    uint64_t file_off;      // first byte (SOI) of this file
    uint64_t rgb_off;       // this image's RGB plane in the workspace (bytes)
    uint32_t entropy_rel;   // first entropy-coded byte
    uint32_t entropy_len;   // bytes up to the EOI marker
    uint32_t coef_block0;   // first block of this image in the coefficient workspace
    uint32_t n_blocks;      // mcu_cols * mcu_rows * blocks_per_mcu
    uint32_t window0;       // first decode window (= workgroup) of this image
    uint32_t n_windows;
    uint32_t rgb_pitch;     // bytes between RGB rows (covers the whole MCU grid)
    uint32_t group0;        // first reconstruction workgroup of this image
    // The groups (runs of MCUs of one MCU row) that reconstruction produces: MCU rows
    // roi_row0 .. + roi_rows - 1, groups roi_gcol0 .. + roi_gcols - 1 of each.  It is what the
    // bilinear taps of the crop window touch, or the whole MCU grid.
    uint16_t roi_row0, roi_rows;
    uint16_t roi_gcol0, roi_gcols;
    uint32_t dht_off[4];    // offset of BITS[16] of: DC luma, AC luma, DC chroma, AC chroma
    uint32_t dht_nval[4];   // number of HUFFVAL bytes that follow the 16 BITS bytes
    uint32_t dqt_off[3];    // offset of the 64 zig-zag ordered table bytes per component
    uint16_t width, height;
    uint16_t mcu_cols, mcu_rows;
    uint16_t restart_interval;  // MCUs, 0 = none
    uint8_t sampling;           // PREP_SAMPLING_*
    uint8_t blocks_per_mcu;
    int32_t status;             // host verdict; kernels skip images that are not PREP_OK
    uint32_t table_slot;        // expanded Huffman tables of this image, or kNoTableSlot
    uint32_t stream0;           // first stream window of this image, and how many: 0 = the stream
    uint32_t n_streams;         // is decode_entropy's alone (restart markers, no table slot)
};
static_assert(sizeof(ImageRec) % 8 == 0, "ImageRec must keep 8-byte alignment in arrays");

// Resize/crop/normalize geometry of one image, computed on the host in double precision
// and handed over in fixed point so that every lane maps coordinates with integer
// arithmetic: source coordinate of output pixel i = (off + i * scale) / 2^kCoordFrac - kCoordBias.
constexpr int kCoordFrac = 30;   // fraction bits (scale < 2^17 and i < 2^16 keep the product in 64 bits)
constexpr int kCoordBias = 16;   // added so that the slightly negative coordinates at the border stay positive
struct ResizeRec {
    uint64_t scale_x, scale_y;  // source pixels per output pixel
    uint64_t off_x, off_y;      // source coordinate of output pixel (0,0), biased
    int32_t src_w, src_h;
    uint32_t src_pitch;
    uint32_t pad_;
    uint64_t src_off;           // byte offset of the source image
};

}  // namespace prep
