// Internal declarations shared by the host API and the gfx950 kernels of librgc.
// Nothing here is visible through the C ABI (include/rgc.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "rgc_tiles.h"

namespace rgc {

// ---------------------------------------------------------------- geometry (compile time)
constexpr int kWaveSize = 64;
constexpr int kBlockThreads = 256;                 // 4 waves per workgroup
constexpr int kWavesPerBlock = kBlockThreads / kWaveSize;
constexpr int kGroupElems = kWaveSize * 4;         // one float4 per lane per step
constexpr int kHistBins = 4096;                    // radix digit of 12 bits (31-bit key = 12+12+7)
constexpr int kCoarseBins = 1024;                  // candidate histogram bins (hinted path)
constexpr int kCoarseRep = 8;                      // replicas of it, to spread same-address atomics
constexpr int kMemberMax = 4096;                   // candidates of one coarse bin ranked in LDS
constexpr uint32_t kKeyMask = 0x7FFFFFFFu;

// Phase a layer has to run at a given launch of the phase kernel.
enum Phase : uint32_t {
  PH_NONE = 0,
  PH_SEL = 1,      // hinted: rank the members of the candidate bin holding the k-th key
  PH_OUT_C = 2,    // hinted: ordered output from the candidate lists
  PH_HIST1 = 3,    // multi-pass: digit-1 histogram over the updated residual (after a miss)
  PH_HIST2 = 4,    // multi-pass: digit-2 histogram
  PH_HIST3 = 5,    // multi-pass: digit-3 histogram
  PH_COUNT = 6,    // multi-pass: per wave-chunk counts of keys > T and == T
  PH_OUT_V = 7,    // multi-pass: ordered compaction from the updated residual
  PH_COLLECT = 8,  // after the first digit: candidate lists from the updated residual, then PH_SEL / PH_OUT_C
  PH_RESTORE = 9,  // dense layers whose hint missed: the entries masked on the strength of the hint go back into residual and
                   // velocity, then PH_HIST1 in the same launch
  PH_EMIT = 10,    // dense layers: the message from the lists, with the k-th entry known
  PH_EMIT_PART = 12,   // tiled calls, larger layers: emit_kernel
  PH_SEL2 = 11,    // dense layers: PH_SEL on the layer's own lists (lists_kernel)
};

constexpr uint32_t kFirstLateLaunch = 4;          // general calls: launches 4 .. 6 only meet the last phases
// Workgroups' worth of candidate lists one workgroup of PH_SEL / PH_OUT_C takes (CompressArgs::list_group:
// kListGroup, or 1 for a call whose workgroups all fit on the device at once, where spreading the lists wins).
constexpr uint32_t kListGroupLog2 = 2, kListGroup = 1u << kListGroupLog2;
// Dense layers: after a call whose hint missed, the layer goes without its hint for a number of calls that
// doubles with every further miss, up to this many.
constexpr uint32_t kDenseBackoffMax = 64;
// Dense layers: the members of the k-th key's coarse bin are appended to this many sub-lists, each with a counter
// of its own (thousands of waves appending through one counter take their turns at ~20 ns each), and what a
// sub-list cannot hold to one more list that can hold them all.
constexpr uint32_t kMemberShards = 16;
constexpr uint32_t kMemberLists = kMemberShards + 1;
constexpr uint32_t kShardStride = 64;    // words between two counters: atomics on one cache line take their turns like atomics on one word

// Tiled calls (see tile_kernel): what select_kernel does with a layer.
constexpr uint32_t kFinishThreads = 1024, kFinishWaves = kFinishThreads / kWaveSize;
constexpr uint32_t kDirectMaxLog2 = 15, kDirectMax = 1u << kDirectMaxLog2;
constexpr uint32_t kTileChunk = 1024;              // elements per wave
constexpr uint32_t kTileElems = kTileChunk * kWavesPerBlock;
constexpr uint32_t kTileSlots = kTileElems / 16;   // slots that a large call on tiles counts on for each tile's list ...
constexpr uint32_t kTileSlotsMost = 480;           // ... and what the lists have where the device has room (see rgc_create()): small calls count
                                                   // on all of them (see counts_on_long_lists() in rgc_api.cpp)
                                                   // (with 512 all lists begin 4 KiB apart: ResNet-50 set 70.0 us, 69.6 this way)
static_assert(kTileSlotsMost % 2u == 0 && kTileSlotsMost <= kTileElems / 8, "16-byte aligned lists; an eighth of the elements is allocated");
constexpr uint32_t kFinishCand = 12288;            // candidates in LDS
constexpr uint32_t kPartTilesMax = 1024;           // lists gather_lists() can take
// A larger layer's parts: kPartTiles tiles (2^20 elements, 2,600 candidates at 0.1 %), at higher densities half as many and again
// until about kPartCand candidates are expected of each, but never more than kPartsMax parts.  A part's candidates are one
// workgroup's work: at 1 % the ResNet-50 set takes 103 us per call, with parts of 2^20 elements whatever the density 143 (2 Mi +
// 0.6 Mi elements: 35 and 84; lines of 3072 and 6144 candidates: within 6 us of this one).
constexpr uint32_t kPartTiles = 256, kPartsMax = 2048, kPartCand = 4096;
static_assert(static_cast<uint64_t>(kPartsMax) * kPartTiles * kTileElems >= (1ull << 31), "any layer has at most kPartsMax parts");
enum LayerKind : uint32_t {
  kLayerBig = 0,       // several workgroups, a message launch of its own
  kLayerLists = 1,     // ended by one workgroup from its lists: the rank its hint is aimed at leaves room in the LDS for twice as many
                       // (with room for half as many more only, a layer whose residual was still building up missed on every call)
  kLayerDirect = 2,    // at most kDirectMax elements: ended by one workgroup from the residual itself, needs no hint
};
constexpr uint32_t kListsTargetMax = kFinishCand / 2;
// A tiled call that counts on more than kTileSlots a list goes back to the general launches for good after a layer's hint has
// missed in this many calls on end: see counts_on_long_lists() in rgc_api.cpp.
constexpr uint32_t kMissRun = 3;
constexpr uint32_t kEmitLaunch = 3;                // tile_kernel is 1, select_kernel 2
constexpr uint32_t kTiledLateLaunch = 4;           // a missed hint: the first digit, in fallback_kernel

// Per call, per layer descriptor (device copy of the caller's rgc_layer plus the tiling).
struct LayerDesc {
  const float* grad;
  float* resid;
  float* mom;
  int32_t* out_idx;
  float* out_val;
  int32_t* out_count;
  uint32_t n;
  uint32_t k;
  uint32_t wc_first;   // first wave-chunk of this layer in the per-wave-chunk arrays
  uint32_t wc_count;   // number of wave-chunks = ceil(n / chunk)
  uint32_t wg_first;   // first workgroup of this layer
  uint32_t wg_count;   // = ceil(wc_count / 4)
  uint32_t grp_first;  // first election-group counter of this layer
  uint32_t hintable;   // one-pass layer: the candidate lists can hold every element from the hinted threshold upwards
  uint32_t margin;     // extra candidates aimed for beyond k
  uint32_t cmax;       // largest candidate total a hint may aim at
  uint32_t target;     // rank the next call's threshold hint is aimed at (2k + margin, dense layers: k + margin)
  uint32_t dense;      // high-density layer (never set together with hintable): with a hint, its streaming pass lists every
                       // candidate in lists of its own and masks those far enough above the hinted threshold at once
  uint32_t mem_cap;    // dense layers: entries of the layer's kMemberShards sub-lists together (a multiple of kMemberShards); the
                       // overflow list behind them holds mem_cap / 4, which is also the most members a call accepts
  uint32_t list_cap;   // dense layers: entries of one wave-chunk's list
  uint32_t kind : 4;         // LayerKind (tiled calls)
  uint32_t part_tiles : 28;  // tiled calls: tiles of a part (one word for both: every workgroup of every launch reads a descriptor,
                             // and 8 bytes more of it cost a call of seven launches 0.4 %)
  uint32_t part_first; // tiled calls: where the layer's parts start in the per-part arrays
  uint64_t mem_first;  // dense layers: where the layer's region of the member pool starts
  uint64_t list_first; // dense layers: where the layer's lists start (wave-chunk c of the layer: list_first + c * list_cap)
};

// Per layer state living in the context (device memory).  Everything but the hint fields is
// rewritten by every call before it is read.
struct LayerState {
  uint32_t next_phase;   // Phase to run ...
  uint32_t next_launch;  // ... at this launch number (general calls 2..6, tiled ones 3..8), in fallback_kernel's launches with kLastPass
  uint32_t done;         // workgroups of the layer that finished the current phase
  uint32_t prefix;       // multi-pass: key bits fixed so far (digits 1 and 2)
  uint32_t k_rem;        // rank of the k-th key inside the current bin (1-based)
  uint32_t T;            // threshold key: the k-th largest key of the layer
  uint32_t r;            // multi-pass: how many keys == T are admitted (lowest indices)
  uint32_t bstar;        // hinted: coarse bin holding the k-th key
  uint32_t nmembers;     // hinted: members appended so far
  uint32_t path;         // 0 hinted one-pass, 1 hint-free multi-pass, 2 miss then multi-pass
  unsigned long long thr;  // hinted: composite (key<<32 | ~idx) of the k-th entry
  // speed hints (never influence results)
  uint32_t hint_valid;
  uint32_t tau;          // candidate threshold key for the next call
  uint32_t shift;        // coarse bin = min((key - tau) >> shift, kCoarseBins - 1)
  uint32_t tau_next;     // being derived during this call
  uint32_t hint_pending; // multi-pass: 0 none found yet / 1 refine in the next digit / 2 final
  uint32_t T_prev;       // threshold key of the previous call (drift estimate), if has_prev
  uint32_t has_prev;
  uint32_t stat_candidates;  // diagnostics of the last call
  uint32_t stat_members;
  uint32_t stat_misses;      // calls so far in which this layer's hint missed (never reset)
  // dense layers (speed only, like the hints)
  uint32_t clip;             // candidates of the coarse bins from this one upwards are sure to be selected: counted, not ranked
  uint32_t dense_backoff;    // calls the layer went without its hint after the last miss
  uint32_t dense_skip;       // calls it still goes without it
  uint32_t cur_tau;          // tau, shift and mask_key as this call's streaming pass used them (the ranking step rewrites
  uint32_t cur_shift;        // the hint for the next call before the output step has read it)
  uint32_t cur_mask_key;
  uint32_t mask_key;         // dense layers: where the k-th key of the next call is expected; its streaming pass masks the candidates
                             // from here upwards at once and the output step puts right what that got wrong
  // tiled calls that count on long lists (speed only)
  uint32_t last_miss;        // CompressArgs::call of the last call in which the hint missed
  uint32_t miss_run;         // calls on end, up to that one, in which it did
};

// Where the kernels of an exactly rounded sum leave their parts (one per workgroup): the running sum
// and the sum of its rounding errors, the flags (digits in use, non-finite terms seen) and, only where
// the flags say so, the part's fixed-point digits.
constexpr int kExactDigits = 20;            // 32 bits each, from 2^-298 upwards: any sum of fp32 terms or of their squares
constexpr size_t kExactWordsPerPart = 3 + kExactDigits;   // 8-byte words of one part
struct ExactParts {
  double* sc;                  // [parts][2]
  unsigned long long* flags;   // [parts]
  long long* digits;           // [parts][kExactDigits]
};
inline ExactParts exact_parts_at(void* base, size_t parts) {
  ExactParts P;
  P.sc = static_cast<double*>(base);
  P.flags = reinterpret_cast<unsigned long long*>(P.sc + 2 * parts);
  P.digits = reinterpret_cast<long long*>(P.flags + parts);
  return P;
}

struct CompressArgs {
  const LayerDesc* layers;
  LayerState* state;
  const uint32_t* wg2layer;
  uint32_t* hist;        // [layers][kHistBins]
  uint32_t* coarse;      // [layers][kCoarseRep][kCoarseBins]
  unsigned long long* members;  // [layers][kMemberMax]
  uint32_t* cand_cnt;    // [wave-chunks]
  uint2* slots;          // [wave-chunks][cap] (float bits, index), ascending index per chunk
  uint32_t* wc_a;        // [wave-chunks] counts, then output offsets
  uint32_t* wc_b;        // [wave-chunks] tie counts, then tie prefixes
  uint2* slots2;         // the lists of the dense layers (LayerDesc::list_first, list_cap; allocated when such a layer is first seen)
  float* slots_u;        // the velocity of every listed element, same layout (restores a masked entry after a miss)
  unsigned long long* members2;  // member pool of the dense layers (LayerDesc::mem_first, mem_cap)
  uint32_t* shard_cnt;   // [layers][kMemberLists][kShardStride] members appended to each sub-list, one counter per 256 bytes
  uint32_t* group_done;  // [election groups] workgroups of the group that finished the current phase
  uint32_t* errflag;     // set non-zero on an internal inconsistency
  uint32_t chunk;        // elements per wave-chunk (multiple of 256)
  uint32_t cap;          // candidate slots per wave-chunk
  uint32_t use_hints;
  uint32_t nesterov;     // momentum correction in its Nesterov form: u = m (u + g), a = (V + u) + g
  uint32_t update_hints;
  uint32_t mask_momentum;
  float m;
  uint32_t launch;       // launch number of the kernel (1..6; in fallback_kernel the number of the launch it stands for)
  const uint2* parts;    // tiled calls: (layer, part of it) of every workgroup of select_kernel, those of the larger layers first
  uint32_t* late;        // [3] fallback_kernel: layers are due, tickets taken, workgroups that have left
  uint32_t late_first;   // the launch numbers fallback_kernel stands for (0: they are launches of their own)
  uint32_t late_last;
  uint32_t sign_xor;     // selection key: see key_of() (0 / 0x80000000: which sign bit keeps an element in the ranking)
  uint32_t sign_filter;  // 0: every element ranks by magnitude; ~0: elements of the other sign rank last (key 0)
  uint32_t reverse;      // the streaming pass takes its workgroups in descending order (and the last pass over dense layers' lists)
  uint32_t past_cache;   // the streaming pass reads and writes residual and velocity past the memory-side cache
  uint32_t list_group;   // workgroups' worth of candidate lists one workgroup of PH_SEL / PH_OUT_C takes (1 or 4)
  const float* grad_scale;   // device word every gradient element is multiplied with first, or null
  ExactParts norm_parts; // [workgroups] parts of the sum of squares (clipping coefficient only)
  const LayerDesc* aims; // null, or [layers] the descriptors whose `target` and `cmax` the multi-pass path aims the next hint at: those
                         // of the tiling that the next call is expected to take, where the two differ
  uint32_t call;         // number of this call among those of its hints
  uint32_t* missing;     // null, or host memory that learns `call` when a layer's hint has missed in kMissRun calls on end
};
// With one of the 4-byte fields between `errflag` and `parts` moved behind them (the others then end 4 bytes earlier, a gap before
// `parts`) the compiler makes select_kernel 73 KB of code instead of 68, and every call of small layers takes 0.2 us more: whoever
// changes that block looks at the size.
static_assert(offsetof(CompressArgs, launch) == 156 && offsetof(CompressArgs, parts) == 160, "select_kernel's code depends on these");

// ---------------------------------------------------------------- threshold binary search selection
struct ThresholdMoments {   // per layer, written by the moments kernel
  float mean;               // mean of |a|
  float max;                // max of |a|
  float span;               // max - mean, rounded
  uint32_t counts_taken;    // counts the bisection took (diagnostics)
  float listed_above;       // searching call: the streaming pass has listed the elements above this magnitude (+inf: none)
  uint32_t lists;           // ... and the lists are all the rest of the call needs
};

struct ThresholdArgs {
  const LayerDesc* layers;
  const uint32_t* wg2layer;
  float* thresholds;        // [layers] the caller's: written by a search, read otherwise
  int32_t* nnz;             // [layers] the caller's, or null: elements above the threshold
  const float* grad_scale;  // device word every gradient element is multiplied with first, or null
  ExactParts sum_parts;     // [workgroups] parts of the sum of |a|
  float* part_max;          // [workgroups] partial maxima of |a|
  uint32_t* counts;         // [wave-chunks] elements above the threshold (then first output positions, if `scanned`)
  uint32_t* wg_counts;      // [workgroups] elements above the threshold (the memory of part_max, which is no longer needed then)
  uint32_t* listed;         // [wave-chunks] elements above the threshold (kept; more than cap: list incomplete)
  uint2* slots;             // [wave-chunks][cap] (float bits, index) of the elements above a reused threshold
  uint32_t cap;             // list slots per wave-chunk
  uint32_t* hist;           // [layers][kHistBins]: four copies of a histogram of 1024 bins
  LayerState* state;        // [layers] and
  uint32_t* group_done;     // [election groups]: the counters of "last workgroup of the layer"
  ThresholdMoments* moments;  // [layers]
  uint32_t chunk;           // elements per wave-chunk
  uint32_t search;          // 1: Algorithm 3 finds the thresholds; 0: they are given
  uint32_t sampled;         // searching call: a sample says what the streaming pass lists (0: it lists nothing)
  uint32_t scanned;         // some layer has more than kOffsetsWgs workgroups: the counts are scanned by a launch of their own
  uint32_t past_cache;      // the first pass reads and writes residual and velocity past the memory-side cache
  uint32_t reverse;         // the first pass takes its workgroups in descending order (and every pass after it the other way)
  uint32_t mask_momentum;
  uint32_t nesterov;
  float m;
};

// Up to this many workgroups a layer, every workgroup that writes a part of the message adds the counts of those before it up by itself
// (268 M elements; 32 KB each at most, 16 on average.  In a layer of 2^31 elements that would be 131 KB each, 8.6 GB together.)  The
// line is a cautious one: a launch that scans / adding, us, thresholds reused and searched: 66 M elements 166 / 157, 206 / 198; 265 M 610 / 580,
// 707 / 676; beyond it 300 M 689 / 657, 796 / 766; 1000 M 2424 / 2223, 2619 / 2506.
constexpr uint32_t kOffsetsWgs = 8192;

// The sample of a searching threshold call: kPieceElems elements from each of up to kSampleThreads places of a layer, and the
// magnitude that threshold_sample_rank() of them exceed.  Lists hold one element in 16 and single ones several times the
// average: layers with a larger share above that magnitude are not listed.
constexpr uint32_t kSampleThreads = 1024, kPieceElems = 16;
constexpr uint32_t threshold_sample_pieces(uint32_t n) {
  return (n + (kPieceElems - 1u)) / kPieceElems < kSampleThreads ? (n + (kPieceElems - 1u)) / kPieceElems : kSampleThreads;
}
constexpr uint64_t threshold_sample_rank(uint32_t n, uint32_t k) {
  return (4ull * k * kPieceElems * threshold_sample_pieces(n) + n - 1u) / n + 24u;
}
constexpr bool threshold_listable(uint32_t n, uint32_t k) {
  const uint64_t samples = static_cast<uint64_t>(kPieceElems) * threshold_sample_pieces(n);
  return 2ull * (4ull * k + 24ull * n / samples) <= n / 16u && threshold_sample_rank(n, k) <= samples;
}

hipError_t launch_threshold_compress(const ThresholdArgs& a, uint32_t num_wgs, uint32_t num_layers, hipStream_t s);

// ---------------------------------------------------------------- decompress
constexpr int kEntryCap = 1024;                   // entries staged per worker batch (generic tiles)
constexpr int kBatchWorkers = 128;                // any number of workers: workers per batch (mask of 4 words)
constexpr int kMaskWords = kBatchWorkers / 32;
constexpr int kQMax = 128;                        // positions hit more than once per batch

struct MsgDesc {                                   // one (worker, layer) message
  const int32_t* idx;
  const float* val;
  uint32_t count;
  uint32_t tab_base;    // first table row of the message's layer
};

struct DecompressLayer {   // one dense buffer
  float* dense;
  uint32_t n;
  uint32_t tiles;         // ceil(n / kTile)
  uint32_t tile_base;     // global id of its first tile
  uint32_t row_base;      // first table row (the layer owns tiles + 1 rows)
  uint32_t pad[2];
};

struct BlockDesc {      // one block of the table-building kernel
  uint32_t msg;         // index into the MsgDesc array
  uint32_t first;       // first entry handled by the block
};

struct DecompressArgs {
  const MsgDesc* msgs;        // [layers][workers]
  const DecompressLayer* layers;
  const BlockDesc* blocks;
  uint32_t* tab;              // [workers][tab_stride]: first entry of each tile; one closing entry per layer
  uint32_t tab_stride;
  uint32_t cus;               // compute units of the device (sizes the persistent grids)
  uint32_t num_workers;
  uint32_t num_layers;
  uint32_t num_blocks;        // (With num_tiles behind num_layers the tile kernel loads the two together, its code moves by eight bytes, and 256
  uint32_t num_tiles;         // messages on the ResNet-50 set take 78.9 us instead of 74.7, added 96.6 instead of 92.0.)
  uint32_t add_to_dst;
  uint16_t tile_log;          // logarithm of the positions a tile
  uint16_t wait_after;        // bit j: a lane waits for its stores after its j-th one of a tile (0: no rule; see stores_at_once())
  uint32_t one_value;         // every message's val points to ONE float that all its entries carry
  float scale;
};
static_assert(offsetof(DecompressArgs, num_blocks) == 48 && offsetof(DecompressArgs, num_tiles) == 52, "the tile kernel's code depends on these");

// Records the text of a failed HIP call for rgc_strerror and returns RGC_EHIP (defined with the host API).
int fail_hip(hipError_t e, const char* what);

// kernel launchers (defined in the .hip files)
hipError_t launch_accumulate(const CompressArgs& a, uint32_t num_wgs, hipStream_t s);
hipError_t launch_collect(const CompressArgs& a, uint32_t num_wgs, hipStream_t s);   // streaming pass of a call with dense layers and hints
hipError_t launch_lists(const CompressArgs& a, uint32_t num_wgs, hipStream_t s);     // its launches 2 and 3
hipError_t launch_phase(const CompressArgs& a, uint32_t num_wgs, hipStream_t s);
hipError_t launch_tiles(const CompressArgs& a, uint32_t num_wgs, hipStream_t s);        // streaming pass of a tiled call
hipError_t launch_select(const CompressArgs& a, uint32_t num_parts, hipStream_t s);
hipError_t launch_emit(const CompressArgs& a, uint32_t num_parts, hipStream_t s);
hipError_t launch_fallback(const CompressArgs& a, uint32_t num_wgs, uint32_t cus, hipStream_t s);
constexpr uint32_t kMeanPartsMax = 128;    // parts per layer at most (rgc_message_means)
hipError_t launch_message_means(const CompressArgs& a, uint32_t num_layers, uint32_t max_k, const ExactParts& parts,
                                float* d_means, hipStream_t s);
hipError_t launch_clip_coefficient(const CompressArgs& a, uint32_t num_wgs, float threshold, float* d_coef, hipStream_t s);
hipError_t launch_poison(LayerState* st, uint32_t num_layers, int mode, hipStream_t s);
hipError_t launch_decompress_table(const DecompressArgs& a, hipStream_t s);
hipError_t launch_decompress_tiles(const DecompressArgs& a, hipStream_t s);
hipError_t launch_decompress_validate(const DecompressArgs& a, uint32_t* status, hipStream_t s);
hipError_t launch_wave_scan_selftest(uint32_t* io, hipStream_t s);

}  // namespace rgc
