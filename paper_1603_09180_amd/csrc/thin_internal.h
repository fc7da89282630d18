// thin_internal.h -- structures shared by the HIP kernels and the host runtime
// of the lambda-leveling library.  Not part of the public ABI (include/thin.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace thin {

// One image as the kernels see it.  buf[0] is the caller's image, buf[1] the
// context-owned twin of the same pitch; round r reads buf[r & 1] and writes
// buf[(r + 1) & 1], so after r rounds the current state is in buf[r & 1].
struct ImgDev {
    void* buf[2];
    int64_t pitch;       // row pitch in elements (both buffers)
    int32_t h, w;
    int32_t dtype;       // 1 = u8, 2 = u16
    uint32_t lambda;
    int32_t adj;         // table: adjacency (0 = (8,4), 1 = (4,8)) + 2 * operator
                         // (0 = lambda-leveling, 1 = lambda-skeleton)
    int32_t tiles_x;     // tile grid of this image
    int32_t tiles_y;
    int32_t tile0;       // index of its first tile in the launch's tile arrays
    int32_t round0;      // launch round at which the image's step 0 starts
    int32_t max_steps;   // parity-step cap (4 * max_passes), INT32_MAX if none
    int32_t slot;        // index of its counters (stable while the image is resident)
    int64_t state0;      // index of its first tile in the per-tile state array
    int32_t fresh;       // serving: admitted since the last step (launch_serve_init)
};

// Per-image counters, written by the kernels with device-scope atomics.
struct ImgCnt {
    unsigned long long lowerings;
    unsigned long long tile_rounds;
    int32_t last_step;   // image-local index of the last step that lowered, -1 if none
    int32_t pad;
    unsigned long long examinations;  // candidates characterised (section 2.1 tests run)
};

// Tiles a round launch visits.  With list == nullptr every tile is visited.
// Otherwise launch round R visits list[(R & 1) * cap + i] for i < count[R % 3]
// (every tile when R == full), and a tile appends the tiles that must be
// visited in round R + 1 (its 3x3 tile block when it lowered something during
// its last 4 steps, itself when it lowered anything) to the other half,
// deduplicated by listed[g] = last round g was queued for.  count[(R + 2) % 3]
// is cleared during round R, before round R + 1 appends to it.
struct WorkList {
    int32_t* list;
    int32_t* count;
    int32_t* grab;     // [6]: next list position to hand out in round R, one counter per
                       // pixel-type launch of the round (grab[2 * (R % 3) + u16]),
                       // cleared like count
    int32_t* listed;
    int32_t cap;
    int32_t full;    // the launch round that visits every tile (-1: none)
};

// Connectivity table entry for an upper-neighbour mask (see thin_topology_table).
//   flags: bit 0 destructible, bit 1 peak and bit 2 end point (skeleton
//          tables only), bits 4..6 T--, bits 8..10 T+
//   comps: byte c = ring mask of the c-th counted lower component
struct alignas(8) TopoEntry {
    uint32_t flags;
    uint32_t comps;
};

// Host-side generation of the 256 entries of one (adjacency, operator) table,
// table index adjacency + 2 * operator.
constexpr int kTables = 4;
void build_topology_table(int adjacency, int op, TopoEntry out[256]);

// The same table as the kernels read it (the device holds 4 x 256 entries):
// indexed by the lower-neighbour mask in the bit order the packed decision
// produces (NW, SW, NE, W, N, S, SE, E from bit 0 on).
//   need:  bits 0..7 how many counted lower components must hold a pixel
//          within lambda of the centre (0: lower whatever their contrast; 8:
//          never), bit 31 set when the centre's own contrast must be within
//          lambda too (skeleton tables: peaks and end points)
//   comps: byte c = mask of the c-th counted lower component, same bit order
struct alignas(8) DecEntry {  // one 64-bit load per lookup
    uint32_t need;
    uint32_t comps;
};
void build_decision_table(int adjacency, int op, DecEntry out[256]);

// Residency variants.  kVarFlags keeps the tile in LDS with a re-examination
// flag byte per pixel, every thread checking fixed cells each step;
// kVarSeeded also starts those flags from the previous round's change
// bitmaps; kVarRegs keeps each thread's 4x4 windows in registers;
// kVarBits keeps the flags as one bit per candidate and class and gathers
// each step's flagged candidates into a dense list; kVarBitsSeeded adds the
// previous round's change bitmaps to kVarBits, kVarRegsSeeded to kVarRegs.
constexpr int kVarFlags = 0, kVarSeeded = 1, kVarRegs = 2, kVarBits = 3, kVarBitsSeeded = 4,
              kVarRegsSeeded = 5;

// Variants that read and write per-tile change bitmaps between rounds.
constexpr bool var_seeded(int v)
{
    return v == kVarSeeded || v == kVarBitsSeeded || v == kVarRegsSeeded;
}
// The same variant without history (for callers that keep none).
constexpr int var_unseeded(int v)
{
    return v == kVarSeeded       ? kVarFlags
           : v == kVarBitsSeeded ? kVarBits
           : v == kVarRegsSeeded ? kVarRegs
                                 : v;
}

// Tiled engine geometry chosen at run time among the compiled variants.
struct TileShape {
    int th, tw, k;   // tile height, width, halo = parity steps per residency
    int nt;          // threads per tile
    int var;         // residency variant (kVar*)
};

// The compiled shape with this tile and halo (nt = 0 when there is none).
TileShape complete_shape(int th, int tw, int k);

// Kernel launchers (thin_kernels.hip).  All enqueue on `stream`.
// Clears counters and tile state; with wl.list, listed[] = -1 and counts 0.
hipError_t launch_init_state(hipStream_t stream, ImgCnt* cnt, int nimg, int32_t* tile_last,
                             int ntiles, int32_t* hist_round, WorkList wl);
// Clears the counters and tile state of the images marked fresh.
hipError_t launch_serve_init(hipStream_t stream, const ImgDev* imgs, int nimg, ImgCnt* cnt,
                             int32_t* tile_state);
// The launch's round is `round`, plus *round_base when round_base is not
// null (graph replays: the same launches serve every chunk of rounds).
// Launch flags of the round kernels.
constexpr int kOneImage = 1;     // every tile belongs to image 0 (no tile_img lookup)
constexpr int kStateIsTile = 2;  // a tile's state index is its tile index
constexpr int kOnlyU8 = 4;       // visit only u8 images (bit-flag variants: u8 LDS tiles)
constexpr int kOnlyU16 = 8;      // visit only u16 images
// A grid of as many blocks as fit on num_cus CUs loops over the tiles.
hipError_t launch_round(hipStream_t stream, TileShape shape, const ImgDev* imgs, ImgCnt* cnt,
                        const int32_t* tile_img, int32_t* tile_last, int ntiles, int round,
                        const DecEntry* lut, int num_cus, uint32_t* hist_bits,
                        int32_t* hist_round, WorkList wl, const int32_t* round_base, int kflags);
// *round_base += n (the last node of a chunk graph).
hipError_t launch_advance(hipStream_t stream, int32_t* round_base, int n);
// Words of one tile's change bitmap (two copies of ntiles bitmaps are needed).
int history_words(TileShape s);
hipError_t launch_step(hipStream_t stream, const ImgDev* img_host, const ImgDev* img_dev,
                       ImgCnt* cnt, int step, const DecEntry* lut);
// Cooperative engine: every round in one launch, grid-wide barriers between
// rounds.  active: 3 zeroed counters; rounds_out receives the rounds run.
hipError_t launch_coop(hipStream_t stream, TileShape shape, const ImgDev* imgs, ImgCnt* cnt,
                       const int32_t* tile_img, int32_t* tile_last, int ntiles,
                       const DecEntry* lut, int32_t* active, int32_t* rounds_out,
                       int max_rounds, int num_cus, uint32_t* hist_bits, int32_t* hist_round,
                       int kflags);
bool tile_shape_supported(TileShape s);

// Small-image engine (k_flow): all steps of its images in one launch, tiles
// exchanging halos through tagged words.
struct FlowImg {
    void* image;
    int64_t pitch;       // row pitch in elements
    int64_t word0;       // its first exchange word
    int32_t h, w;
    int32_t dtype;       // 1 = u8, 2 = u16
    uint32_t lambda;
    int32_t adj;         // table index (adjacency + 2 * operator)
    int32_t tiles_x, tiles_y;
    int32_t tile0;       // its first tile
    int32_t slot;        // its counters; ImgCnt.pad is its mark
    int32_t ctl0;        // its ring of kFlowRing vote words
};
struct FlowShape {
    int th, tw, k, nt;
};
struct FlowRun {
    const FlowImg* imgs;
    const int32_t* tile_img;  // tile -> image, null with one image
    int ntiles;
    int grid;
    ImgCnt* cnt;
    const DecEntry* lut;
    int32_t* ctl;
    uint64_t* exch;
    int max_polls, max_rounds;
    int vote_every;           // rounds between votes (a power of two)
};
constexpr int kFlowNext = 0, kFlowAbort = 16;  // control words
constexpr int kFlowCtl = 32;                   // first vote ring
constexpr int kFlowRing = 1024;
constexpr int kFlowPolls = 1 << 17;            // of a wait, unless set
// Rounds of an image, far beyond what one takes (every round but the last
// lowers something; a spiral corridor through n x n pixels takes n * n / 16),
// and within what the kernel's round tags and step numbers count.
constexpr int kFlowMaxRounds = 1 << 24;
constexpr int kFlowMaxSide = 500;              // tiles across or down an image
constexpr int kFlowRunning = 0, kFlowStable = 1, kFlowGivenUp = 2;  // marks
// Exchange words of an image: two copies of one (u8) or two (u16) per 2x2 cell.
inline int64_t flow_words(int64_t h, int64_t w, int dtype)
{
    return 2 * dtype * ((h + 1) / 2) * ((w + 1) / 2);
}
// Blocks of the shape that are resident on the device together.
int flow_capacity(FlowShape s, int num_cus);
hipError_t launch_flow(hipStream_t stream, FlowShape s, const FlowRun& r);
// Clears counters, control and exchange words; writes *one to r.imgs when not null.
hipError_t launch_flow_init(hipStream_t stream, const FlowRun& r, int nimg, int nctl,
                            int64_t exch_words, const FlowImg* one);

// Gradient front-end (gradient.hip): float32 coefficients of Deriche's
// recursive smoothing (a0..a3) and derivative (d1, d2) filters, shared
// feedback (b1, b2) and the steady states of the four recursions for a
// constant input of 1 (the edge rule).
struct GradCoef {
    float a0, a1, a2, a3, d1, d2, b1, b2, s_plus, s_minus, d_plus, d_minus;
};
// Column pass, row pass and output pass on `stream`; scratch holds 8 h*w
// float planes; mag (nullable) receives the float magnitude, h*w contiguous.
constexpr int kGradPlanes = 8;
hipError_t launch_gradient(hipStream_t stream, const void* src, int64_t src_pitch, int src_dtype,
                           int h, int w, float* scratch, void* dst, int64_t dst_pitch,
                           int dst_dtype, float* mag, GradCoef co, float gain, int num_cus);
// Pixel work-list engine (k_worklist): one block per image runs parity
// steps one after the other, examining only the candidates whose 3x3
// changed since their last examination.
struct WlImg {
    void* image;          // the image state, updated in place
    const void* prev;     // init 1: the state one tiled round earlier (same pitch)
    uint32_t* gbits;      // pending bitmaps in global memory (4 * lh * lww words), or null
    int64_t pitch;        // row pitch in elements
    int32_t h, w;
    int32_t dtype;        // 1 = u8, 2 = u16
    uint32_t lambda;
    int32_t adj;          // table index (adjacency + 2 * operator)
    int32_t step0;        // global index of the first step to run
    int32_t max_steps;    // step cap (global index), INT32_MAX if none
    int32_t init;         // 0: every interior candidate pending; 1: those whose 3x3 differs
                          // between image and prev
    int32_t slot;         // counter slot
    int32_t pad;
};
constexpr int kWlThreads = 1024;
constexpr int kWlListCap = 2048;      // entries per candidate list
constexpr int kWlLdsWords = 8192;     // pending-bitmap words kept in LDS (32 KiB)
// Pending-bitmap words of an image (4 classes of ceil(h/2) rows of
// ceil(ceil(w/2)/32) words).
inline int64_t wl_bitmap_words(int64_t h, int64_t w)
{
    return 4 * ((h + 1) / 2) * ((((w + 1) / 2) + 31) / 32);
}
// One block per image; steps_out[i] receives the global index one past the
// last step image i ran.  gbits selects the variant with the pending bitmaps
// in global memory (every image of the launch must have gbits set then).
hipError_t launch_worklist(hipStream_t stream, const WlImg* imgs, int nimg, int dtype,
                           bool gbits, ImgCnt* cnt, const DecEntry* lut, int32_t* steps_out);

// Writes descriptor d to *dst on `stream` (a kernel argument, so no host
// buffer has to outlive the call).
hipError_t launch_set_desc(hipStream_t stream, ImgDev* dst, const ImgDev& d);

// The static scratch array of the no-allocation entry point (noalloc.hip):
// its size, and the device address of the copy on `device`, looked up once
// per device (the caller makes `device` current).
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
hipError_t noalloc_scratch(int device, void** out);

// Every compiled shape: writes up to cap of them to out, returns the count.
int compiled_shapes(TileShape* out, int cap);
int round_blocks_per_cu(TileShape s);

}  // namespace thin
