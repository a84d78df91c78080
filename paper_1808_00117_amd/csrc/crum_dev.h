// Internal device-side structures and kernel launch interface of libcrum.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace crum {

// Diff unit: min(page, 2^unit_shift_max) bytes, unit_shift_max in 12..14
// (default 14).  A wave compares one unit per step with 64 lanes x 16-byte
// loads, i.e. unit/1 KiB loads per array per lane.
constexpr uint32_t kUnitShiftDefault = 14;
// CRC piece: pages larger than this are split across waves and combined.
constexpr uint32_t kPieceShift = 16;  // largest pack piece: 64 KiB
constexpr uint32_t kPieceShiftMin = 12;
// Default piece: 16 KiB, between what snapshots and rollbacks like best.  Us a pass
// with pieces of 4, 16 and 64 KiB: a first snapshot of 1 GiB in 2 MiB pages 428, 438
// and 453, 8 GiB in 64 KiB pages with 9 % dirty 2765, 2783 and 2789, 64 MiB of them
// 61, 61 and 67; a verified rollback of 805 MB in 64 KiB pages 497, 485 and 480.
constexpr uint32_t kPieceShiftDefault = 14;
// Flags of launch_pack.
constexpr int kPackNtStore = 1;  // the image is written with non-temporal stores
constexpr int kPackNtLoad = 2;   // pages are read with non-temporal loads
constexpr uint32_t kNoBad = 0xFFFFFFFFu;

// One region of the flattened page space (host-built, uploaded per call).
// Page indices are global across all requests of a launch; each request
// starts at a multiple of 64 pages so that bitmap words never straddle
// requests.
struct DevRegion {
    const uint8_t* cur;
    uint8_t* shadow;     // NULL: no baseline
    uint64_t len;
    uint64_t first_page; // global page index of page 0
    uint64_t first_unit; // global diff-unit index of unit 0
    uint64_t id;
    uint32_t page_shift; // log2 page size
    uint32_t req;        // request index
    uint32_t unit_shift; // log2 diff unit = min(page_shift, unit_shift_max)
    uint32_t flags;      // bit 0: copy dirty pages into the shadow
};
static_assert(sizeof(DevRegion) == 64, "DevRegion layout");

constexpr uint32_t kReqShadow = 1;  // some region has a shadow

// One request (one image) of a launch.
struct DevRequest {
    uint64_t first_word;   // first bitmap word (global)
    uint64_t n_words;
    uint64_t n_pages;      // pages of the request (unpadded G)
    uint64_t first_region; // index into the region table
    uint32_t n_regions;
    uint32_t flags;        // kReq* bits
    uint64_t data_off;     // image prefix bytes
    uint64_t seq;
    uint32_t page_shift;
    uint32_t init_fix;     // CRC constant for one page (see gf2.h)
};
static_assert(sizeof(DevRequest) == 64, "DevRequest layout");

// Per-request results written on the device.
struct DevReqOut {
    int32_t code;
    uint32_t first_bad;
    uint64_t n_dirty;
    uint64_t total_pages;
    uint64_t image_bytes;
    uint64_t slot_base;  // global slot of the request's first packed page
    uint64_t img_base;   // byte offset of the request's image in staging
    // header / image-check kernels: CRC shares of crcs_crc and meta_crc,
    // arrivals, and a flag or count; zero before those kernels run (the final
    // scan clears them for a snapshot, the host for a restore)
    uint32_t acc[4];
};
static_assert(sizeof(DevReqOut) == 64, "DevReqOut layout");

// Launch-wide counters written on the device.
struct DevGlobal {
    uint64_t total_dirty;    // sum of D over requests
    uint64_t staging_used;   // bytes of staging the images occupy
    int32_t code;            // CRUM_OK or CRUM_ENOSPC (any request) / CRUM_EFORMAT
    uint32_t fmt_bad;        // restore: image check failed
    uint32_t crc_bad;        // restore: lowest failing slot, kNoBad if none
    uint32_t bad_call;       // on-demand restore: first call that found a bad page
    uint64_t running;        // dirty pages counted by the scans so far
    uint64_t img_next;       // 4 KiB-aligned staging offset for the next image
    uint64_t pad[2];
};
static_assert(sizeof(DevGlobal) == 64, "DevGlobal layout");

// The tables of a call with one request and few regions, passed as a kernel
// argument; scratch holds them in this layout too.
constexpr uint32_t kArgRegions = 16;
struct CallTables {
    DevRequest req;
    DevReqOut out;
    DevGlobal glob;
    DevRegion regs[kArgRegions];
};

// CRC constants held in device memory:
// z4k[i][b] = (b << 8i) * x^(8 * 4096): byte i of a state carried through 4 KiB
// of zeros (staged into LDS); xp[i] = x^(8 * 2^i); xb[k][i] = x^(8 * 4096 *
// 256^k * i); xr[i] = x^(8 * 4i).
// mf[4t + p][l]: lane l's FP4 operand of the pack's CRC matrix for 1 KiB step
// t of a 4 KiB batch and bit plane p; col[k][n][j] = (n << 4k) * x^(128 (31 - j)):
// nibble k of column j's state carried past the columns after it (LDS).
struct CrcTables {
    uint32_t z4k[4][256];
    uint32_t xp[64];
    uint32_t xb[3][256];
    uint32_t xr[1024];
    uint32_t col[8][16][32];
    uint32_t mf[16][64][4];
    uint32_t init_fix[31];  // host: crc_init_fix of a page of 2^i bytes
    uint32_t pad;
};

// Clock words of a timed diff launch (see launch_diff).
constexpr uint32_t kStampSlots = 64;
constexpr uint32_t kStampLine = 16;  // 128 bytes
constexpr uint32_t kStampWords = kStampLine * (1 + kStampSlots);

enum PackMode { kModePack = 0, kModeVerify = 1, kModeScatter = 2, kModePull = 3 };

struct LaunchShape {
    int diff_blocks;   // largest grid of the diff kernel (256-thread blocks)
    int pack_blocks;   // persistent grid of the pack/verify/scatter kernels
};

// Slot range of a pack launch: [lo, hi) given on the host, or, when `bounds`
// is non-null, read on the device as [chunk ? bounds[chunk-1] : 0, bounds[chunk]).
struct SlotRange {
    uint64_t lo, hi;
    const uint64_t* bounds;
    uint32_t chunk;
    uint64_t max_slots;  // upper bound on hi - lo (grid sizing)
    uint32_t backward = 0;  // scatter: last slot first
};

// Runs of consecutive slots laid end to end, for launches over several at once
// (on-demand restores).
constexpr uint32_t kMaxRuns = 16;
struct RunList {
    uint32_t n = 0;
    uint32_t call = 0;            // number of the session call they belong to
    uint64_t first[kMaxRuns] = {};  // first slot of run r
    uint64_t end[kMaxRuns] = {};    // slots in runs 0..r
    const uint8_t* host = nullptr;  // read here (the host image, mapped by the device)
};

// Pinned host words that a scan writes itself (each may be null), so that the
// host need not wait for a copy or an event: used = the staging bytes the images
// occupy; count = the running total of dirty pages, with kCountNoSpace when a
// table's one request does not fit.
constexpr uint64_t kCountNoSpace = 1ull << 63;
struct HostNote {
    uint64_t* used = nullptr;
    uint64_t* count = nullptr;
};

// Where a snapshot's bitmap words come from: the region table and the diff's
// unit flags (regs null: the bitmap is there already).
struct FlagSource {
    const DevRegion* regs = nullptr;
    uint32_t n_regs = 0;
    const uint8_t* unit_flags = nullptr;
};

// Up to three copies of one launch: 8-byte aligned, whole 8-byte words.
struct CopyList {
    const void* src[3] = {};
    void* dst[3] = {};
    uint64_t bytes[3] = {};
    CopyList& add(int k, const void* s, void* d, uint64_t n)
    {
        src[k] = s;
        dst[k] = d;
        bytes[k] = n;
        return *this;
    }
};

// Kernel launchers (crum_kernels.hip).  All enqueue on `s`.
// Copies the pieces of `list` from or to pinned host memory; with done (pinned),
// one workgroup copies and then stores 1 there.
hipError_t launch_begin(const CopyList& list, uint64_t* done, hipStream_t s);
const CrcTables& crc_tables();  // the constants, in host memory
// cand (may be null): bitmap over global pages; pages whose bit is clear are
// flagged clean without being read (they are known to equal their shadow).
// stamp (may be null): kStampWords words, below any clock value at first (zeroed
// once): the wall clock at the launch's start in word 0, and the latest end of its
// workgroups as the largest of words kStampLine, 2 * kStampLine, ...
// blocks: largest grid.
// group 2 or 4: each wave takes that many consecutive units (as many 4 KiB
// units of a region read as one span); other values: one unit per wave.
hipError_t launch_diff(const DevRegion* regs, uint32_t n_regs, uint64_t u0, uint64_t u1,
                       uint8_t* unit_flags, int blocks, int nontemporal, int prio,
                       hipStream_t s, const uint64_t* cand = nullptr,
                       uint64_t* stamp = nullptr, int group = 1);
// Scans bitmap words [w0, w1) continuing glob->running; writes the new running
// total to *bounds_out when non-null.  With fs, the words are first formed from
// the diff's unit flags: inside the scan kernel when the range is short, else by a
// k_bitmap launch.  With `final`, also fills the results of
// requests [q0, q1) (whose words must all have been scanned), lays their
// images out from glob->img_next and applies the capacity check: a group that
// does not fit, and every later group, gets CRUM_ENOSPC.  With `list`, also
// writes the slot list of the words (as launch_list): inside the scan kernel
// when the range takes one pass, else by a launch_list behind it.
hipError_t launch_scan(uint64_t* bitmap, uint64_t w0, uint64_t w1, uint32_t* prefix,
                       uint64_t* bounds_out, int final, const DevRequest* reqs, uint32_t q0,
                       uint32_t q1, DevReqOut* out, DevGlobal* glob, uint64_t capacity,
                       int restore_mode, uint32_t* list, hipStream_t s, const FlagSource& fs,
                       const HostNote& note = HostNote{});
// launch_diff over units [0, u1) of a call's tables, which it also stores at `to`.
hipError_t launch_diff_first(const CallTables& t, CallTables* to, uint32_t n_regs, uint64_t u1,
                             uint8_t* unit_flags, int blocks, int nontemporal, int prio,
                             hipStream_t s, int group);
hipError_t launch_list(const uint64_t* bitmap, const uint32_t* prefix, uint64_t w0, uint64_t w1,
                       uint32_t* list, hipStream_t s);
// Pack, verify and scatter work on (slot, piece) items: a page of 2^ps bytes
// is cut into pieces of 2^min(ps, piece_shift) bytes, np_shift is log2 of the
// largest piece count per slot in the launch, and finalize combines the piece
// CRCs of pages larger than one piece.  Pack updates the shadows of regions
// whose flags bit 0 is set.  unit_flags (pack only, may be null): the diff's
// per-unit flags of the same page space (4-byte aligned, padded to whole
// words); units flagged clean are then read from the shadow.  nt: kPackNt*
// bits.  update_shadow (scatter only): pages go to the shadows as well.  runs
// (may be null; verify, scatter, pull): the slots, instead of range.  A scatter
// of a range also does what launch_restore_finish does, with h_status.
hipError_t launch_pack(int mode, const DevRegion* regs, uint32_t n_regs, const DevRequest* reqs,
                       DevReqOut* out, const uint32_t* list, SlotRange range,
                       uint32_t np_shift, uint32_t piece_shift, const uint8_t* unit_flags,
                       uint8_t* staging, uint32_t* crc_out, uint32_t* partials,
                       const CrcTables* tabs, DevGlobal* glob, int blocks, hipStream_t s, int nt,
                       int update_shadow = 0, const RunList* runs = nullptr,
                       void* h_status = nullptr);
hipError_t launch_finalize(int mode, const DevRegion* regs, uint32_t n_regs,
                           const DevRequest* reqs, const DevReqOut* out, const uint32_t* list,
                           SlotRange range, uint32_t np_shift, uint32_t piece_shift,
                           const uint32_t* partials, uint32_t* crc_out, uint8_t* staging,
                           DevGlobal* glob, const CrcTables* tabs, hipStream_t s,
                           const RunList* runs = nullptr);
// Workgroups per request for launch_header and launch_restore_check, from
// the request's region count, bitmap words and (a bound on) its CRC count.
uint32_t header_blocks(uint64_t n_regions, uint64_t n_words, uint64_t n_crcs);
// `blocks` workgroups per request of [q0, q1).  Requests with ENOSPC get only
// their prefix (header, table, bitmap), and only when it fits within
// `capacity`.  h_status (device-mapped pinned memory, may be null): gets the
// first request's crum_status.
hipError_t launch_header(const DevRegion* regs, const DevRequest* reqs, uint32_t q0, uint32_t q1,
                         uint32_t blocks, DevReqOut* out, const uint64_t* bitmap,
                         const uint32_t* crcs, uint8_t* staging, uint64_t capacity,
                         const CrcTables* tabs, hipStream_t s, void* h_status = nullptr);
// Resets the launch-wide counters (graph-safe: a kernel, not a memset).
hipError_t launch_plan_init(DevGlobal* glob, hipStream_t s);
// Compact per-request results: {code, first_bad, n_dirty, total_pages,
// image_bytes, image_offset} (40 bytes each) for requests [0, n).
hipError_t launch_plan_status(const DevReqOut* out, uint32_t n, uint8_t* dst, hipStream_t s);
// The image checks that need its bytes (bitmap population and unused bits,
// zero pads, crcs_crc, meta_crc), `blocks` workgroups per request; a failure
// sets glob->fmt_bad.  out[q].acc must be zero.
hipError_t launch_restore_check(const DevRequest* reqs, uint32_t n_reqs, uint32_t blocks,
                                DevReqOut* out, const uint8_t* staging, const CrcTables* tabs,
                                DevGlobal* glob, hipStream_t s);
hipError_t launch_restore_finish(DevReqOut* out, uint32_t n_reqs, DevGlobal* glob,
                                 hipStream_t s, void* h_status = nullptr);

}  // namespace crum
