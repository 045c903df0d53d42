// Internal constants and layout helpers of the gfx950 Pici library.  Host and
// device code of the library share this header; nothing outside the library
// includes it.
#pragma once
#include <stdint.h>

namespace spccl {

constexpr uint32_t kMagic = 0x49434950u;        // "PICI"
constexpr uint64_t kHeaderBytes = 48;
constexpr uint64_t kNnzUnknown = ~0ull;
constexpr uint32_t kTileElems = 4096;           // a 64 x 64 virtual tile
constexpr uint32_t kWave = 64;                  // CDNA wavefront
constexpr uint32_t kWavesPerBlock = 4;          // one tile per wave
constexpr uint32_t kBlockThreads = kWave * kWavesPerBlock;
constexpr uint32_t kTilesPerPart = kWavesPerBlock;   // look-back partition = one block
constexpr uint32_t kStageBytes = 7168;          // LDS staging per wave (an fp32 tile up to 7/16 full in one go)

constexpr int kFmtDense = 0, kFmtPici = 1, kFmtCoo = 2;
constexpr int kKindArray = 0, kKindStream = 1;
constexpr int kF32 = 0, kBF16 = 1;

// Workspace: a control block, then one 64-bit look-back word per partition.
struct WsCtrl {
    uint32_t status;     // sticky device status (first error wins)
    uint32_t pad[63];
};
static_assert(sizeof(WsCtrl) == 256, "control block is 256 bytes");
constexpr uint64_t kWsFlagsOffset = sizeof(WsCtrl);

__host__ __device__ inline uint64_t elem_bytes(int dtype) { return dtype == kBF16 ? 2 : 4; }
__host__ __device__ inline uint64_t num_tiles(uint64_t n) { return (n + kTileElems - 1) / kTileElems; }
__host__ __device__ inline uint64_t off_I(uint64_t n) { return kHeaderBytes + 512ull * num_tiles(n); }
__host__ __device__ inline uint64_t off_A(uint64_t n) {
    return (off_I(n) + 4ull * (num_tiles(n) + 1) + 15ull) & ~15ull;
}
__host__ __device__ inline uint64_t pici_bytes(uint64_t n, int dtype, uint64_t nnz) {
    return off_A(n) + nnz * elem_bytes(dtype);
}
__host__ __device__ inline uint64_t dense_msg_bytes(uint64_t n, int dtype) {
    return kHeaderBytes + n * elem_bytes(dtype);
}
// COO message: header, J (nnz 32-bit flat indices, increasing) at 48, zero
// pad to 16 bytes, V (nnz values) at coo_off_V(nnz).
__host__ __device__ inline uint64_t coo_off_V(uint64_t nnz) { return (kHeaderBytes + 4ull * nnz + 15ull) & ~15ull; }
__host__ __device__ inline uint64_t coo_bytes(int dtype, uint64_t nnz) {
    return coo_off_V(nnz) + nnz * elem_bytes(dtype);
}
constexpr uint64_t kPartElems = (uint64_t)kTilesPerPart * kTileElems;

__host__ __device__ inline uint64_t num_parts(uint64_t n) {
    uint64_t T = num_tiles(n);
    uint64_t p = (T + kTilesPerPart - 1) / kTilesPerPart;
    return p ? p : 1;
}

// The second pass of a two-pass Pici sink sums the partitions' aggregates per
// chunk of kPlaceChunk partitions; each chunk's sum has a look-back word of its
// own, after the partitions' words.
constexpr uint32_t kPlaceChunk = 256;
__host__ __device__ inline uint64_t num_place_chunks(uint64_t nparts) {
    return (nparts + kPlaceChunk - 1) / kPlaceChunk;
}
// look-back words of a workspace for n elements: one per partition, one per chunk
__host__ __device__ inline uint64_t flag_words(uint64_t n) {
    const uint64_t p = num_parts(n);
    return p + num_place_chunks(p);
}

// A fresh 30-bit epoch for the look-back words of one launch (host).
uint32_t next_epoch();

// Source kinds of the tile pipeline.
enum SrcKind { SRC_NONE = 0, SRC_DENSE = 1, SRC_PICI = 2, SRC_COO = 3 };

// A reduce / codec operand as the kernels see it.
struct DevOperand {
    const uint8_t* hdr;    // message header, or nullptr for a raw array
    const uint8_t* data;   // raw array base, or the message base for Pici / COO
    uint64_t cap;          // capacity of the message buffer in bytes
    const uint64_t* idx;   // COO: idx[t] = epoch << 32 | first entry of tile t (T + 1 words, k_coo_index),
                           // or nullptr: search J
    uint32_t idx_epoch;    // the epoch of this call's index words; a tile whose words carry another searches J
};

// One rank's send of one step of a ring decided on the device (Sec. IV-C): its
// sigma0, the tracked sparsity before this send's own count (a Pici send is
// measured), its count (Pici) and its format.
struct RingRank {
    double sigma0, sigma_prev;
    uint64_t nnz;
    int32_t fmt, pad;
};

struct PiciSinkArgs {
    DevOperand a, b;
    uint8_t* out;          // output message base
    uint64_t n;
    uint64_t T;
    uint32_t nparts;
    uint32_t epoch;        // tags this call's look-back words (unique per launch)
    WsCtrl* ctrl;
    uint64_t* flags;
    uint8_t* slots;        // two-pass mode: one worst-case slot of compacted values per partition
    uint32_t* idx_slots;   // COO output: one worst-case slot of flat indices per partition
    uint64_t* nnz_out;     // the output's count once it is known, beside the header (nullptr: not wanted)
    RingRank* nnz_rows;    // a batch: rank r's count goes to nnz_rows[r].nnz (nullptr: not wanted)
};

struct DenseSinkArgs {
    DevOperand a, b;
    uint8_t* out_hdr;      // nullptr for an ARRAY output
    uint8_t* out;          // output element base
    uint64_t n;
    uint64_t T;
    WsCtrl* ctrl;
};

constexpr int kMaxGatherParts = 64;
struct GatherArgs {
    DevOperand part[kMaxGatherParts];
    uint8_t* out;          // element base of part 0 of this launch
    uint64_t n;            // elements per part
    uint64_t T;
    WsCtrl* ctrl;
};

// Sliced streams: slot q of a stream holds elements [kSliceElems q, ...) as
// an ordinary message; one block (4 tiles) produces or consumes one slice.
constexpr uint64_t kSliceElems = kPartElems;
__host__ __device__ inline uint64_t num_slices(uint64_t n) { return (n + kSliceElems - 1) / kSliceElems; }
__host__ __device__ inline uint64_t slice_slot_bytes(int dtype) {
    const uint64_t p = pici_bytes(kSliceElems, dtype, kSliceElems), d = dense_msg_bytes(kSliceElems, dtype);
    return p > d ? p : d;
}

enum SlicedOp { kSlicedCompress = 0, kSlicedReduceToSliced = 1, kSlicedReduceToDense = 2, kSlicedExpand = 3 };

struct SlicedArgs {
    const uint8_t* a;      // dense input array, or a sliced stream (expand, copy)
    const uint8_t* b;      // sliced input stream, or nullptr
    uint8_t* out;          // sliced output stream, or dense output array
    uint64_t n;            // elements
    uint64_t slot;         // bytes per slot
    double thresh;         // a produced slice is dense iff its sparsity <= thresh (tracked: iff the
                           // tracker's estimate <= thresh)
    WsCtrl* ctrl;
    double* track;         // per slice: sigma0, sigma_prev (nullptr: decide on the measured sparsity)
    int32_t track_step;    // 0: the first send (sigma0 := measured); 1: a later one (Eq. 7 estimate)
    uint8_t* fmt_out;      // per slice: the format produced (nullptr: not recorded)
    uint8_t* fwd;          // expand: the stream is also written here, for the next hop (nullptr: not)
};

// One sliced ring step for up to kMaxBatchRanks virtual ranks in a single
// launch (grid y = rank): rank r's arguments are base with its own dense or
// source pointer a[r], output out[r] and forwarded stream fwd[r], its
// threshold, and strided received streams, trackers and format records.
constexpr int kMaxBatchRanks = 32;
struct SlicedBatch {
    SlicedArgs base;
    const uint8_t* a[kMaxBatchRanks];
    uint8_t* out[kMaxBatchRanks];
    uint8_t* fwd[kMaxBatchRanks];
    double thresh[kMaxBatchRanks];
    uint64_t b_stride;               // bytes between ranks
    uint64_t track_stride;           // doubles between ranks
    uint64_t fmt_stride;             // bytes between ranks
};

// One step of the canonical ring for a batch of virtual ranks in a single
// launch (grid y = the rank's place in the batch): each rank's operands,
// output, look-back words and value slots; sizes, the epoch, capacities and
// the status word are the launch's base arguments, shared.  An operand
// pointer replaces the base operand's (a message keeps its header-to-data
// offset); a null b leaves the base's b.
struct RankBatch {
    const uint8_t* a[kMaxBatchRanks];
    const uint8_t* b[kMaxBatchRanks];
    uint8_t* out[kMaxBatchRanks];
    uint8_t* flags[kMaxBatchRanks];     // the rank's look-back words (zeroed once per collective)
    uint8_t* slots[kMaxBatchRanks];     // the rank's value slots (two-pass Pici sink)
    const RingRank* gate;               // the place pass: only ranks whose send in this row is Pici (nullptr: all)
    int32_t rank[kMaxBatchRanks];       // the rank of each entry
};

// The launches of a device-decided ring.
enum RingLaunch { kRingFirst = 0, kRingStep = 1, kRingGather = 2 };

// The state of a device-decided ring: P ranks a row, one row per send (step 0
// .. P - 2 of the reduce-scatter, then the all-gather's at row P - 1).
struct RingArgs {
    RingRank* rows;
    uint64_t slot_bytes;
    uint64_t m;               // elements per message
    int32_t P, step;
    int32_t last;             // the step that reduces into the output
    double intra, inter, ag;  // the policy's thresholds
    int32_t ranks_per_node, adaptive;
};

__host__ __device__ inline RingRank* ring_row(const RingArgs& a, int step) { return a.rows + (uint64_t)step * a.P; }

__host__ __device__ inline bool rank_skipped(const RankBatch& rb, uint32_t j) {
    return rb.gate && rb.gate[rb.rank[j]].fmt != kFmtPici;
}

__host__ __device__ inline DevOperand rebase(DevOperand o, const uint8_t* p) {
    if (o.hdr) {
        o.data = p + (o.data - o.hdr);
        o.hdr = p;
    } else {
        o.data = p;
    }
    return o;
}

__host__ __device__ inline PiciSinkArgs rank_sink(PiciSinkArgs g, const RankBatch& rb, uint32_t r) {
    g.a = rebase(g.a, rb.a[r]);
    if (rb.b[r]) g.b = rebase(g.b, rb.b[r]);
    g.out = rb.out[r];
    g.flags = reinterpret_cast<uint64_t*>(rb.flags[r]);
    g.slots = rb.slots[r];
    if (g.nnz_rows) g.nnz_out = &g.nnz_rows[rb.rank[r]].nnz;
    return g;
}

__host__ __device__ inline SlicedArgs batch_rank(const SlicedBatch& b, uint32_t r) {
    SlicedArgs g = b.base;
    g.a = b.a[r];
    if (g.b) g.b = b.base.b + r * b.b_stride;
    g.out = b.out[r];
    g.fwd = b.fwd[r];
    g.thresh = b.thresh[r];
    if (g.track) g.track = b.base.track + r * b.track_stride;
    if (g.fmt_out) g.fmt_out = b.base.fmt_out + r * b.fmt_stride;
    return g;
}

}  // namespace spccl
