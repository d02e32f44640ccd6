// fk_internal.hpp -- records shared by the host runtime and the kernels.
//
// The host turns a chain descriptor into these plain records once per plan
// (compute ops) and once per run (batch items); the kernels read them with
// uniform (scalar) loads.
#pragma once
#include <stdint.h>

namespace fk {

enum : int32_t {
    RD_PLAIN = 0,
    RD_CROP_RESIZE = 1,
    RD_CROP_NEAREST = 2,
    RD_NV12 = 3,
    RD_NV12_RESIZE = 4,
};
// read kinds with an output size of their own (not the ROI's)
constexpr bool rd_resizes(int rk) { return rk == RD_CROP_RESIZE || rk == RD_CROP_NEAREST || rk == RD_NV12_RESIZE; }
// read kinds whose kernels use the fp32 scales w/ow and h/oh
constexpr bool rd_bilinear(int rk) { return rk == RD_CROP_RESIZE || rk == RD_NV12_RESIZE; }
enum : int32_t { DT_U8 = 0, DT_F16 = 1, DT_F32 = 2, DT_F64 = 3 };
enum : int32_t { LY_PACKED = 0, LY_PLANAR = 1, LY_STATS = 2 };
// Kernel selection only: a planar write, or a packed one of several channels,
// from pixel-strided lanes (bilinear reads on launches of at least
// kStridedMinPixels output pixels).
enum : int32_t { LY_PLANAR_PX = 3, LY_PACKED_PX = 4 };

// Normalised compute op codes.  SUB becomes ADD of the negated constant
// (IEEE x - y is x + (-y)), CVT disappears (fp32 from the read on), swaps
// move to the read, and in the contracted mode a MUL followed by ADD/SUB
// becomes FMA.  LOOP sends execution back over the `span` records before
// it until they have run `count` times.
enum : int32_t { OPC_MUL = 0, OPC_ADD = 1, OPC_DIV = 2, OPC_FMA = 3, OPC_LOOP = 4 };

constexpr int kUnitPx = 4;       // output pixels per unit: one 16-byte planar fp32 store
constexpr int kMaxBlock = 1024;  // largest block the kernels accept
constexpr int kWave = 64;        // CDNA wavefront

struct OpRec {          // 48 bytes
    int32_t code;
    int32_t span;       // LOOP: body records just before this one
    int32_t count;      // LOOP: runs of the body in all (>= 1)
    int32_t pad;
    float a[4];         // MUL/ADD/DIV constant per channel, or FMA multiplier
    float b[4];         // FMA addend per channel
};

// The op list as the kernels run it (lower_ops): OpSeg records up to a
// SEG_END, then a pool of constants in the running value's type V (fp32, or
// fp64 for a chain with an fp64 write).  MUL, ADD and FMA records all become
// multiply-adds, so a stretch of them is one loop with no branch on the op:
// x * k is fma(x, k, -0.0) and x + k is fma(x, 1, k), each with the same one
// rounding (and the same signed zero) as the op itself.
enum : int32_t {
    SEG_FMA1 = 1,  // n records, constants shared by the channels: V m, a
    SEG_FMAC = 2,  // n records, constants per channel: V m[4], a[4]
    SEG_FMAR = 4,  // one record per channel (as SEG_FMAC), run `reps` times
    SEG_DIV = 8,   // one division (DivRec32 / DivRec64), run `reps` times
    SEG_LOOP = 16, // the n segments before it run `reps` times in all
    SEG_END = 32,  // after the last segment
};
struct OpSeg {          // 16 bytes
    int32_t kind;
    int32_t n;
    uint32_t off;       // the segment's constants, bytes from the list's start
    int32_t reps;
};
static_assert(sizeof(OpSeg) == 16, "OpSeg layout");

// Division by a constant d, correctly rounded without the general division
// sequence, where every dividend of the group is zero, infinite, NaN or
// has a biased exponent of at least E (thr = (E << exponent shift) - 1 in
// the high word shifted left by one); other groups take the general division.
//  fp32: (float)((double)x * y) with y = RN64(1 / d).  The product is within
//  2^-51.9 of x / d, and a quotient of two 24-bit numbers that is not
//  subnormal lies at least 2^-49 from every rounding boundary, so it rounds
//  as x / d does; E keeps the quotient normal.
//  fp64: fma(x, zh, x * zl) with zh + zl = 1 / d to 2^-106.  d has 24 bits,
//  so the quotient lies at least 2^-78 from every rounding boundary; E keeps
//  it above 2^-900.  v_div_fixup sets the zeros, infinities and NaN.
struct DivRec32 {       // 64 bytes
    double y[4];
    float d[4];
    uint32_t thr;
    uint32_t pad[3];
};
// The compile-time normalise chain's division record, in its constant table
// after the chain's seven constants.
constexpr int kDivRecOffset = 32;
struct DivRec64 {       // 112 bytes
    double zh[4], zl[4], d[4];
    uint32_t thr;
    uint32_t pad[3];
};
static_assert(sizeof(DivRec32) == 64 && sizeof(DivRec64) == 112, "division record layout");

// Item flags.
enum : int32_t {
    IF_SRC_VEC = 1,     // source rows 4-byte aligned: unit loads as dwords
    IF_CONTIG = 4,      // plain read of whole frame rows stored back to back, under
                        // 2^31 pixels: one row of ow * oh pixels, unit u starting
                        // u * 4 pixels after row y
    IF_SMALL_FRAME = 8, // frame below 4 GiB, rows below 16 MiB: 32-bit row offsets
};

struct ItemRec {        // 64 bytes: one batch slot's parameters
    uint64_t src;       // frame base address (device)
    uint64_t dst;       // output base address (device)
    int64_t pitch;      // frame row pitch in bytes
    int32_t x, y, w, h; // region of interest in the frame
    int32_t ow, oh;     // output size
    float sx, sy;       // crop+resize scales w/ow and h/oh (fp32)
    uint16_t fw, fh;    // frame size in pixels (bounds of window reads)
    int32_t flags;      // IF_*
};
static_assert(sizeof(ItemRec) == 64, "ItemRec layout");

struct RunHeader {      // per-run header read by the kernel (graph-friendly)
    int32_t n_items;
    uint32_t total_tiles;
    int32_t pad[2];
};

// Small batches ride in the kernel arguments instead of a device table:
//  - full:    ItemRec[inl_n] at inl[0..], uint32 tile_begin[inl_n + 1] at
//             inl[kInlineTileBegin..] (inl_n <= kInlineItems);
//  - compact: items sharing one frame geometry, one output size and a
//             constant output stride: an ItemRec template at inl[0..64) (item
//             0) and one record per item from inl[64] on; item b owns tiles
//             [b * inl_tiles_per_item, (b + 1) * inl_tiles_per_item).  The
//             record is the least that differs: CF_ROI of one frame, the ROI;
//             CF_POINT of one frame read 1:1, its corner (every ROI has the
//             output's size); CF_FRAME of several frames, frame and ROI.
#ifndef FK_INLINE_BYTES
#define FK_INLINE_BYTES 2560
#endif
constexpr int kInlineBytes = FK_INLINE_BYTES;
constexpr int kInlineItems = (kInlineBytes - 4) / 68 < 32 ? (kInlineBytes - 4) / 68 : 32;
constexpr int kInlineTileBegin = kInlineItems * 64;
struct Roi16 {
    uint16_t x, y, w, h;
};
struct Point16 {
    uint16_t x, y;
};
struct FrameRoi16 {
    uint64_t src;
    Roi16 roi;
};
static_assert(sizeof(Point16) == 4 && sizeof(Roi16) == 8 && sizeof(FrameRoi16) == 16 &&
                  __builtin_offsetof(FrameRoi16, roi) == 8,
              "the kernels read these records as dwords");
enum : int32_t { CF_NONE = 0, CF_ROI = 1, CF_POINT = 2, CF_FRAME = 3 };
constexpr int compact_items(int form)
{
    return (kInlineBytes - 64) / (form == CF_POINT ? (int)sizeof(Point16)
                                  : form == CF_FRAME ? (int)sizeof(FrameRoi16) : (int)sizeof(Roi16));
}
constexpr int kCompactItems = compact_items(CF_ROI);  // 312 (624 points, 156 frames)

// Stats write: a block's partial result for one channel.
struct StatPartial {    // 16 bytes
    float mn, mx;
    double sum;
};

// Stats write: a batch slot's output is covered by at most kStatSlots
// blocks (each striding over the item's tiles); each leaves one partial per
// channel, and a second kernel combines each item's partials.
constexpr int kStatSlots = 512;
// Partials a stats plan holds (slots over a whole batch); a batch of n
// items gives each at most kStatCapacity / n slots, and at most the
// resident grid's blocks / n, so that each block walks several tiles.
constexpr int kStatCapacity = 65536;

// Kernel arguments (by value, the only kernel argument, so it starts the
// kernarg segment).  Device table layout of one run:
//   RunHeader | ItemRec[max_batch] | uint32 tile_begin[max_batch + 1]
struct KArgs {
    const RunHeader *hdr;
    const ItemRec *items;
    const uint32_t *tile_begin;
    const OpSeg *ops;      // run-time tier op list (device), lowered, up to its SEG_END
    const float *consts;   // compile-time tier constants (device)
    int32_t pad0;
    int32_t swap;          // net BGR<->RGB swap applied at the read
    int32_t strict;        // compile-time tier: 1 = no contraction
    int32_t loop_count;    // compile-time loop chain: pairs to run
    int32_t inl_n;         // > 0: the run's items are in `inl`
    int32_t inl_compact;   // compact form: CF_*
    uint32_t inl_total_tiles;
    uint32_t inl_tiles_per_item;  // compact form
    int64_t inl_dst_stride;       // compact form: bytes between item outputs
    StatPartial *st_part;  // stats write: one partial per (slot, channel)
    alignas(16) uint8_t inl[kInlineBytes];
};

// Kernel families.
enum : int32_t {
    FAM_RUNTIME = 0,       // any chain: run-time op list
    FAM_NORMALIZE = 1,     // crop+resize u8x3 -> swap,cvt,mul,sub,div -> planar f32
    FAM_MULADD = 2,        // plain u8x3 -> cvt, N x (mul, add) -> packed f32
    FAM_MULADD_LOOP = 3,   // plain u8/f32 x1/x3 -> [cvt,] mul, add, loop(2, P) -> packed f32
    FAM_F64 = 4,           // plain read -> run-time op list in fp64 -> fp64 packed/planar
};

// Kernel lookup (defined by the kernel translation units).  Returns the
// host-side kernel handle to pass to hipLaunchKernel, or nullptr if the
// combination is not built.
const void *kernel_runtime(int read_kind, int in_dt, int channels, int out_dt, int layout,
                           int coarsen);
// strided: pixel-strided lanes (launches of at least kStridedMinPixels
// output pixels), else 4-pixel units
const void *kernel_normalize(int coarsen, int strict, int strided);
constexpr uint64_t kStridedMinPixels = 1u << 20;
// The same for fp16 and fp32 frames, whose pixels hold up to 16 loaded dwords
// a lane (units and strided lanes: 15 fp32 crops to 213 x 273 x 4 13.5 and
// 10.1 us, 6 to 224 x 224 x 3 6.3 and 6.0, 6 fp16 ones 6.5 and 6.2; one
// channel is level, 5.5 and 5.6 for 10 fp32 crops; at 2^17 all are level).
constexpr uint64_t kStridedMinPixelsWide = 1u << 18;
// crop+resize of a u8 frame with the tapped rows staged in LDS
const void *kernel_normalize_lds(int coarsen, int strict);
// LDS of a staged-row gather block of T threads (dynamic shared memory)
constexpr uint32_t lds_gather_bytes(uint32_t T) { return T * 128u < 65536u ? T * 128u : 65536u; }
const void *kernel_muladd(int n_ops, int coarsen, int strict);
// plain read of in_dt elements -> run-time op list in fp64 -> fp64 write
const void *kernel_f64(int in_dt, int channels, int layout, int coarsen);
const void *kernel_muladd_loop(int in_dt, int channels, int coarsen, int strict);
const void *kernel_loop_px(int in_dt, int channels, int coarsen, int strict);
// The compile-time loop chain runs per pixel (k_loop_px, a tile = T*K
// pixels) from this many pairs on; shorter loops keep the 4-pixel unit.
constexpr int kLoopPxMinPairs = 32;
const void *kernel_stats(int read_kind, int in_dt, int channels, int coarsen);
// stats write of a plain u8 read with no arithmetic after the cast
const void *kernel_stats_u8(int channels, int coarsen);
const void *kernel_stats_final(int channels);

}  // namespace fk
