// gravac.hip - Top-k + error-feedback gradient compression for MI355X (gfx950).
//
// Implements the C ABI of include/gravac.h.  The path follows GraVAC (arxiv 2305.12201):
// error feedback (Sec. III-B), Top-k sparsification at a compression factor (Sec. II-C),
// residual update (Alg. 1), compression gain for several candidate CFs (Sec. III-B
// equation, Alg. 1 gain steps), layerwise mode and decompression (Sec. III-A).
//
// Design in one paragraph.  Keys are the binary32 bit patterns of |acc|, so magnitude order is
// unsigned-integer order.  A small stratified sample of acc gives, per candidate CF, a bracket
// [lo, top) of keys that holds the k-th largest key with a statistical safety margin.  ONE streaming
// pass then reads grad and residual, writes acc back as the provisional residual, sums acc^2, and for
// every CF counts (and sums the energy of) the entries above the bracket and histograms the entries
// inside it.  The few entries inside some bracket go, in index order, into a per-sub-tile bracket list
// (zeros are only counted); the entries that can belong to the committed selection go into a
// per-sub-tile candidate list, unless the sub-tile is mostly candidates, in which case the emit step
// reads it again from the residual.  Everything after the pass works on those lists: locate the
// histogram bin that holds the k-th largest, gather the few keys of that bin, resolve the exact key,
// scan the counts and emit the message in ascending index order while zeroing the selected residual
// slots.  If a sampled bracket turns out wrong the segment is redone by a route that cannot fail: a bin
// too coarse and too full to resolve is binned again inside itself from the bracket lists; a k-th
// largest outside the bracket is found from a 2048-bin histogram of the top key bits of all elements,
// after which the lists are collected again.  A flat tensor of at most DIRECT_MAX elements is sampled
// whole, which gives the bin itself, and needs neither the bracket's histogram nor those routes.
// Results are identical on every route; only the number of passes over memory differs.
//
// Units of work.  A tile is TW consecutive elements; the streaming pass gives each of its SUB
// sub-tiles to one 64-lane wavefront, which owns that sub-tile's slots of the list arrays, so
// ordered compaction needs no communication between wavefronts and no list can overflow.  The list
// kernels give a wavefront a unit: a tile, or in calls of few tiles half or a quarter of one.  Cross-tile
// results (histograms, output offsets) are combined at kernel boundaries, and no workgroup waits for
// another, except on the exact routes, which run inside the plan step, and where a direct call's emit step
// cuts a full bin again (wide_resolve): there the workgroups wait for each other over counters in the
// workspace.  Such a workgroup works on one segment, waits only once every
// chunk of it has been claimed, hence only for workgroups that are running and wait for nobody before
// they have arrived, and gives up after a number of polls (wait_for_all).  Global atomics complete at a
// rate of roughly one per cache line per 10 ns on this part, so what takes many of them is spread: the
// bracket histogram and the gather lists' fill counts exist in REP copies (picked from the sub-tile,
// tile or workgroup number), the counts above the brackets lie on 64 lines.  The others are few: a
// tile's counts added to those of its 64-tile group, the exact routes' histograms (one add per workgroup
// and bin, or per wavefront and bin) and queue counters, the status record.

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include "gravac.h"
#include "gravac_profile.h"

namespace {

#ifndef GV_TW
#define GV_TW 8192
#endif
constexpr int TW = GV_TW;           // elements per tile (unit of the list kernels)
#ifndef GV_SUB
#define GV_SUB 8
#endif
constexpr int SUB = GV_SUB;         // sub-tiles per tile: the streaming pass gives one wavefront a sub-tile
constexpr int TS = TW / SUB;        // elements per sub-tile
constexpr int WG = 256;             // threads per workgroup of the streaming kernels
constexpr int WAVES = WG / 64;
#ifndef GV_LWG
#define GV_LWG 256
#endif
constexpr int LWG = GV_LWG;         // threads per workgroup of the list kernels (refine, emit)
constexpr int LWAVES = LWG / 64;
constexpr int ROW = 256;            // elements one wavefront touches per load (64 lanes x float4)
constexpr int ROWS = TS / ROW;      // rows of a sub-tile: all of them are in flight together
static_assert(TS % ROW == 0 && ROWS == 4, "a sub-tile is four rows");
#ifndef GV_DENSE
#define GV_DENSE 384
#endif
constexpr uint32_t DENSE_SUB = GV_DENSE;  // a full sub-tile with at least this many candidates keeps no candidate list:
                                          // the emit step reads its 1024 elements again (4 KB read + 4 KB written, what
                                          // about 400 listed candidates cost in list traffic and scattered stores)
constexpr uint32_t DENSE_BIT = 0x80000000u;  // flag of such a sub-tile in cand_cnt
constexpr uint32_t LONG_WALK = 256;   // a tile with at least this many listed entries is walked sub-tile by sub-tile
#ifndef GV_NT
#define GV_NT 1                     // non-temporal hints on the streaming loads and stores
#endif
// A flat Top-k call of at most this many elements is direct: the sampling kernel histograms all of them, so the brackets are
// the bins that hold the k-th largest, what lies above them is known, and the pass gathers their entries itself; the plan and
// refine steps are left out.
#ifndef GV_DIRECT
#define GV_DIRECT 524288
#endif
constexpr int64_t DIRECT_MAX = GV_DIRECT;
constexpr int REP = 8;              // copies of the bracket histogram and of the gather lists
constexpr int NBIN = 2048;          // bins of the bracket / refine / coarse histograms
constexpr uint32_t OVF = NBIN - 1;  // bins 0 .. OVF - 1 cover the bracket; bin OVF stands for everything above it
// Bins of the sample histogram, in key order: SCOARSE bins of 2^19 keys (16 per octave, 4.4 % in magnitude) from
// |x| = 2^-48 up to 2^16 (smaller magnitudes share the first, larger ones the last), except that a window of SWIN octaves
// is cut into bins of 2^15 keys (256 per octave, 0.27 %).  A bracket's ends are bin edges, so a bin's entries are what it
// has too many.  (4096 bins of 1.1 % everywhere: at CF 10 the bracket held three times the statistically needed entries.)
constexpr int SBIN = 4096;
constexpr uint32_t SCSHIFT = 19, SFSHIFT = 15;
constexpr uint32_t SEXP0 = 79, SOCT = 64;      // exponent field of 2^-48, octaves
constexpr uint32_t SWIN = 12, SWIN_ABOVE = 2;  // octaves of the window, and how many of them lie above the largest of 256 samples
// (The look at the 256 elements costs a 1 MiB bucket 0.4 of 33.4 us.  A window given by the host for small tensors, 2^-14
// to 2^-2, spared it for magnitudes of 1e-4 to 1e-1 alone: 33.0 us for Normal(0, 1e-3), but 38.4 for 1e-7 and 37.4 for 1;
// equal bins of 1.1 %, 33.9 for all.)
constexpr uint32_t SKEY0 = SEXP0 << 23;
constexpr uint32_t SCOARSE = SOCT << (23 - SCSHIFT), SFINE = SWIN << (23 - SFSHIFT), SLESS = SWIN << (23 - SCSHIFT);
constexpr uint32_t SUSED = 1 + SCOARSE + SFINE - SLESS;   // bins in use: the first is the key 0 alone
static_assert(SUSED <= (uint32_t)SBIN && (uint64_t)SKEY0 + ((uint64_t)SOCT << 23) <= 0x7F800000ull, "inside the finite keys");
constexpr int SGRP = 8;             // the sample bins in SGRP groups: a workgroup of the threshold kernel each (up to 32 tensors)
constexpr int RGRP = 64;            // ... and in RGRP groups: a wavefront of the bracket kernel each (flat calls)
constexpr int SAMPLE_BLOCK = 1024;  // samples per workgroup of the sampling kernel
constexpr int SAMPLE_MAX = 65536;   // samples of a flat tensor at most (unless k n is large, see SAMPLE_MAX_FLAT)
constexpr int SAMPLE_MAX_SEG = 32768;  // layerwise: samples per tensor at most (a tensor of up to twice that is read whole)
constexpr int SAMPLE_MAX_FLAT = 524288;  // flat mode, a large k: see sample_count
constexpr int DENSE_ROUNDS = 4;          // ... whose sample blocks are up to DENSE_ROUNDS * SAMPLE_BLOCK samples each
constexpr int DENSE_BLOCKS = 128;        // ... so that there are at most this many of them
constexpr int LCAP = 4096;          // keys a gather list can hold
constexpr int MAXCF = GRAVAC_MAX_CF;
constexpr double ZMARGIN = 5.0;     // safety margin of the sampled rank, in standard deviations
constexpr uint32_t CTILES = 64;     // units per partial sum of the units' counts (csum)
constexpr int FINE = 2, MIDDLE = 4; // sub-tiles per wavefront of the list kernels where a tile each leaves the chip idle (units_per_tile)
constexpr int XQ_WORDS = 8;         // a segment's work queue in the plan step: chunks claimed, then chunks done per phase
constexpr int XQ_WIN = XQ_WORDS;    // ... and behind it the first key of its sample histogram's window
constexpr int XQ_LINE = 32;         // words between two segments' queues: a cache line
constexpr int BND_WORDS = 32;       // words of a segment's brackets, a cache line: lo, hi, mid and (direct calls) mode per CF
static_assert(4 * GRAVAC_MAX_CF <= BND_WORDS, "a bracket per CF");
constexpr uint32_t WAIT_POLLS = 1u << 26;  // polls after which a workgroup of the plan step gives up on the others: at least
                                           // half a minute, where the longest wait of a call is milliseconds
constexpr uint32_t WAIT_POLLS_TEST = 256;  // ... and under GRAVAC_FLAG_STALL_FALLBACK
constexpr uint32_t NONE = 0xFFFFFFFFu;
constexpr uint32_t KEY_END = 0x80000000u;  // one past the largest key

enum : uint32_t { MODE_RESOLVED = 0, MODE_GATHER = 1,
                  MODE_WIDE = 2,   // a direct call's bin that is too full to gather or too wide: cut again by the emit step
                  MODE_FAIL = 3 };
// What the plan step found for a segment, the heaviest kind over its CFs:
//   FAIL_TIES    the bin that holds the k-th largest is at most 2^11 keys wide and too full to gather (a mass of equal
//                values): it is counted key by key, from the bracket lists;
//   FAIL_NARROW  the bin is known but too coarse and too full to resolve: only the CFs concerned are binned again, inside
//                that bin, from the bracket lists (no pass over the gradient);
//   FAIL_FULL    the k-th largest lies outside the bracket (or there was none): acc is read again.
enum : uint32_t { FAIL_NONE = 0, FAIL_TIES = 1, FAIL_NARROW = 2, FAIL_FULL = 3 };
// where a call's brackets come from
enum : uint32_t { BOUNDS_SAMPLED = 0, BOUNDS_RANDOM = 1, BOUNDS_FORCED = 2,
                  BOUNDS_FIXED = 3 };  // the threshold sparsifier: the caller gives the threshold, nothing is searched for

// Selection state of one (segment, CF).
struct CfState {
    uint32_t k;         // entries to select
    uint32_t lo;        // first key of the bracket histogram's bin 0
    uint32_t s;         // bin = (key - lo) >> s
    uint32_t mode;      // MODE_*
    uint32_t base;      // first key of the bin that holds the k-th largest
    uint32_t span;      // a key lies in that bin iff 0 <= key - base <= span
    uint32_t above;     // number of keys above that bin
    uint32_t c;         // number of keys in that bin
    uint32_t tau;       // key of the k-th largest (valid once resolved)
    uint32_t need;      // how many keys equal to tau are selected (lowest indices first)
    uint32_t cnt_gt;    // number of keys greater than tau
    uint32_t top;       // the pass over the gradient has counted keys >= top as above the bracket (KEY_END: none)
    uint32_t pad[4];
};
static_assert(sizeof(CfState) == 64, "CfState layout");

struct SegState {
    uint32_t fail;    // FAIL_*: whether a bracket failed and the segment takes an exact route, and which
    uint32_t pz;      // sparse sub-tiles: the first pass has stored +0 instead of acc for keys >= pz: the upper end of the
                      // committed CF's bracket, above which an entry is selected unless the bracket fails (NONE: none)
};

struct Status {
    int any_fail;
    int n_fail;
    int error;
    int n_seg;
    int n_narrow;             // segments of n_fail that were only binned again from their bracket lists
    int count;                // threshold sparsifier: entries at or above the threshold (written by the scan)
    int n_wide;               // 1: a direct call whose emit step has cut a full bin again (MODE_WIDE)
    int pad;
};

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
// The same at any address of a float: a gfx950 load or store of 16 bytes needs no more than 4-byte alignment, and a tensor
// of a layerwise call starts anywhere (38 million elements as 387 tensors, three in four of which start off a multiple of four
// elements: 153 us, with their elements one by one 213).
typedef v4f v4fu __attribute__((aligned(4)));
typedef v4i v4iu __attribute__((aligned(4)));

// One tensor of a layerwise call.
struct SegInfo {
    int64_t begin, end;      // element range in the flat gradient
    int64_t koff;            // offset of the segment's message in out_idx / out_val
    uint32_t tile0, tile1;   // tile range
    uint32_t samp0;          // first sample block
    uint32_t samp_cnt;       // samples taken
    uint32_t small;          // 1: at most SMALL_MAX elements, handled by one workgroup out of LDS: no tiles, no samples
    uint32_t rep;            // copies of the segment's bracket histograms and gather lists: REP for a large tensor, else 1
    uint32_t pool0;          // its first copy block in hist1 / list_* / list_cnt (n_cf * rep consecutive blocks, CF-major)
    uint32_t wg0, wgs;       // its first workgroup in the emit step, and how many
    uint32_t pad[1];
};
static_assert(sizeof(SegInfo) == 64, "SegInfo layout");

struct Params {
    const float* grad;       // gradient; in single-source mode the values of the level-1 message
    float* res;              // residual (in: leftover, out: acc with the selection zeroed); null in single-source mode
    const float* acc;        // where acc can be re-read after the streaming pass: res, or grad in single-source mode
    const int32_t* map_idx;  // single-source mode: index of every source element in the dense gradient (else null)
    float* restore;          // single-source mode: dense residual that gets the unselected values back (or null)
    int64_t n_restore;       // its length
    int single;              // 1 = single-source mode (second-level compression of a message)
    int random;              // 1 = Random-k: the order is that of a keyed priority of the index, not of |acc|
    int no_commit;           // 1: nothing is removed from the residual (it keeps acc); the caller commits a message later
    uint32_t bounds_from;    // BOUNDS_*
    uint32_t direct;         // 1: the sample is the whole tensor, and its histogram says which bin holds the k-th largest
    uint32_t fixed_key;      // BOUNDS_FIXED: the key of the caller's threshold; entries with key >= fixed_key are kept
    uint32_t wait_polls;     // polls after which a workgroup of the plan step stops waiting for the others
    uint32_t wait_extra;     // arrivals it waits for beyond those that will come: 0 (1 under the testing flag)
    uint32_t rk_s0, rk_s1;   // Random-k: the two 31-bit keys (from the seed)
    int64_t n;
    int n_seg;  // >= 1
    int n_cf;
    int commit;
    int64_t total_out;        // pairs the call emits
    uint32_t n_tiles;
    uint32_t n_sample_blocks;
    // layerwise tables in the workspace (unused when n_seg == 1)
    const SegInfo* segs;           // [n_seg] built on the host
    const uint32_t* ktab;          // [n_seg][n_cf] built on the host
    const uint32_t* sblock_seg;    // [n_sample_blocks] segment of every sample block, built on the host
    uint32_t* tseg;                // [n_tiles] segment of every tile, filled by threshold_kernel
    // the same for one flat tensor
    uint32_t flat_k[MAXCF];
    uint32_t flat_samples;
    // workspace
    Status* status;
    CfState* st;         // [n_seg][n_cf]
    SegState* seg;       // [n_seg]
    uint32_t* bnd;       // [n_seg][BND_WORDS] the bracket of every CF: first key, one past the last key (at most KEY_END), the key
                         // the sample puts the k-th largest at (NONE: no estimate)
    uint32_t* hist1;     // [copy blocks][NBIN] bracket histograms: REP copies per CF of a large tensor, one otherwise
    uint32_t* ovfc;      // [n_seg][n_cf][64][32] counts above the bracket (the histogram's last bin), spread over
                         // 64 cache lines; word 0 of each line is used
    uint32_t* xq;        // [n_seg][XQ_LINE] the plan step's work queue of every segment (XQ_*)
    uint32_t* coarse;    // [n_seg][NBIN] histogram of key >> 20 (exact route)
    uint32_t* list_key;  // [copy blocks][LCAP] gather lists: key ... (before they are filled: the exact routes' histograms)
    uint32_t* list_tile; //                          ... unit ...
    float* list_val;     //                          ... and value (written for Random-k only) of the listed entries
    uint32_t* list_cnt;  // [copy blocks][32] fill counts of the gather lists, one cache line each
    uint32_t* samp_hist; // [n_sample_blocks][SBIN / 2] sample histograms, two 16-bit counts per word
    uint16_t* samp_above;  // [n_sample_blocks][RGRP] the block's samples above each group of SBIN / RGRP bins
    uint32_t* cand_cnt;  // [n_tiles][SUB] listed candidates of every sub-tile (| DENSE_BIT: none listed, the sub-tile is read again)
    uint32_t* brk_cnt;   // [n_tiles][SUB] bracket-list entries of every sub-tile (| zeros counted instead of listed << ZERO_SHIFT)
    uint32_t* ovn;       // [n_tiles][SUB][n_cf] entries of the sub-tile above CF j's bracket
    double* ovs;         // [n_tiles][SUB][n_cf] ... and their sum of acc^2
    // (units: tiles, or half or quarter tiles in calls of few; see units_per_tile)
    uint32_t* tg0;       // [units] entries of the unit above the committed CF's located bin
    uint32_t* tin;       // [units] entries of the unit inside that bin
    // a call with a scan step:
    uint32_t* toff;      // [n_tiles] offset of the tile's output inside its segment's message
    uint32_t* ttake;     // [n_tiles] how many of the tile's entries equal to tau(commit) are selected
    uint32_t* tsel;      // [n_tiles] pairs the tile emits
    // ... and one without (null otherwise):
    uint64_t* csum;      // [units / CTILES, rounded up][8] sums of tg0 (high half) and tin over CTILES units: word 0 of a cache line
    uint32_t n_csum;     // their number
    uint32_t* wseg;      // [workgroups of the emit step] the segment of each (layerwise; filled by threshold_kernel)
    double* ssd;         // [n_tiles][SUB] sum of acc^2 of every sub-tile
    double* ssd_t;       // [units] sum of acc^2 of the unit
    double* sss;         // [units][n_cf] sum of acc^2 over the unit's keys above CF j's located bin
    int32_t* cand_idx;   // [n_tiles][SUB][TS] candidate list: sub-tile j of tile u owns the slots from (u*SUB + j)*TS
    float* cand_val;     // [n_tiles][SUB][TS]
    uint32_t* brk_key;   // [n_tiles][SUB][TS] bracket list: keys ...
    float* brk_val;      // [n_tiles][SUB][TS] ... and values (written for Random-k only)
    // outputs
    int32_t* out_idx;
    float* out_val;
    int64_t* out_count;
    double* out_stats;
};

// ---------------------------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ bool is_flat(const Params& p) { return p.n_seg == 1; }
__device__ __forceinline__ int64_t seg_begin(const Params& p, int t) { return is_flat(p) ? 0 : p.segs[t].begin; }
__device__ __forceinline__ int64_t seg_end(const Params& p, int t) { return is_flat(p) ? p.n : p.segs[t].end; }
__device__ __forceinline__ uint32_t seg_tile0(const Params& p, int t) { return is_flat(p) ? 0u : p.segs[t].tile0; }
__device__ __forceinline__ uint32_t seg_tile1(const Params& p, int t) { return is_flat(p) ? p.n_tiles : p.segs[t].tile1; }
__device__ __forceinline__ uint32_t seg_k(const Params& p, int t, int j) { return is_flat(p) ? p.flat_k[j] : p.ktab[t * p.n_cf + j]; }
__device__ __forceinline__ int64_t seg_koff(const Params& p, int t) { return is_flat(p) ? 0 : p.segs[t].koff; }
__device__ __forceinline__ int tile_seg(const Params& p, uint32_t u) { return is_flat(p) ? 0 : (int)p.tseg[u]; }
__device__ __forceinline__ bool seg_small(const Params& p, int t) { return !is_flat(p) && p.segs[t].small != 0u; }
// Copy blocks: one holds a copy of a (segment, CF)'s bracket histogram (NBIN words of hist1), a gather list (LCAP
// slots of list_*) and its fill count (a cache line of list_cnt).  Copy r of (t, j) is block seg_block(p, t, j) + r.
__device__ __forceinline__ uint32_t seg_rep(const Params& p, int t) { return is_flat(p) ? (uint32_t)REP : p.segs[t].rep; }
__device__ __forceinline__ size_t seg_block(const Params& p, int t, int j)
{
    return is_flat(p) ? (size_t)j * REP : (size_t)p.segs[t].pool0 + (size_t)j * p.segs[t].rep;
}

// A direct call's histograms of a bin that is cut again, one per round: in the values of CF j's gather lists, which Top-k does
// not use.
constexpr uint32_t WIDE_ROUNDS = 3;   // 11 bits each, of up to 31
__device__ __forceinline__ uint32_t* wide_hist(const Params& p, int j, uint32_t round)
{
    static_assert(WIDE_ROUNDS * NBIN <= REP * LCAP && WIDE_ROUNDS * 11 >= 31, "the rounds' histograms fit, and resolve any key");
    return (uint32_t*)p.list_val + (size_t)j * REP * LCAP + round * NBIN;
}

__device__ __forceinline__ uint32_t key_of(float a) { return __float_as_uint(a) & 0x7FFFFFFFu; }

// Bin of the sample histogram a key falls into, and the keys a bin spans; w0: first key of the window (the start of an
// octave, not of the lowest).
__device__ __forceinline__ uint32_t sample_bin(uint32_t key, uint32_t w0)
{
    const uint32_t c0 = (w0 - SKEY0) >> SCSHIFT;
    const uint32_t d = key < SKEY0 ? 0u : key - SKEY0, c = d >> SCSHIFT;
    const uint32_t f = key - w0;                       // (wraps below the window)
    if (f < (SWIN << 23)) return 1u + c0 + (f >> SFSHIFT);
    const uint32_t cc = c < SCOARSE - 1u ? c : SCOARSE - 1u;
    return cc < c0 ? cc + (key != 0u ? 1u : 0u) : 1u + cc + SFINE - SLESS;   // (the window does not start at the lowest octave: 0 < c0)
}
// first key of bin b; the next bin's is one past its last key
__device__ __forceinline__ uint32_t sample_bin_first(uint32_t bin, uint32_t w0)
{
    const uint32_t c0 = (w0 - SKEY0) >> SCSHIFT;
    if (bin >= SUSED) return KEY_END;
    if (bin <= 1u) return bin;
    const uint32_t b = bin - 1u;
    if (b >= c0 && b < c0 + SFINE) return w0 + ((b - c0) << SFSHIFT);
    return SKEY0 + ((b < c0 ? b : b - (SFINE - SLESS)) << SCSHIFT);
}
__device__ __forceinline__ uint32_t sample_bin_end(uint32_t b, uint32_t w0) { return sample_bin_first(b + 1u, w0); }

// The bracket histogram of a CF whose bracket is [lo, hi): bin (key - org) >> s, the shift the smallest with which bins
// 0 .. OVF - 1 reach hi, and top the first key past them (KEY_END if they reach past the largest key).  org is lo, unless
// the bracket starts at zero: then bin 0 is the key 0 alone.  Zeros are the one value that a gradient is likely to have a
// mass of, and a k-th largest among them is resolved with the bin.
__device__ __forceinline__ void bracket_bins(uint32_t lo, uint32_t hi, uint32_t& s, uint32_t& org, uint32_t& top)
{
    const uint32_t span = hi > lo ? hi - lo : 0u;
    s = 0;
    org = lo;
    if (span == 0u) { top = lo; return; }  // an empty bracket: every key from lo on counts as above it
    const uint32_t last = lo == 0u ? OVF - 2u : OVF - 1u;
    s = span >> 11 ? 21u - (uint32_t)__clz((int)span) : 0u;   // span >> s < 2^11
    if ((span >> s) > last) ++s;
    if (lo == 0u) org = 1u - (1u << s);    // (wraps: (0 - org) >> s is 0, (1 - org) >> s is 1)
    const uint64_t t = (uint64_t)lo + ((uint64_t)OVF << s) - (lo == 0u ? (1u << s) - 1u : 0u);
    top = t >= (uint64_t)KEY_END ? KEY_END : (uint32_t)t;
}

// Where bin b of a 2048-bin histogram lies: neighbouring bins in different 128-byte lines, 64 lines in turn.  An atomic
// takes its L2 channel about 4 ns (a million adds to all lines of eight copies take 35 us, to the lines of 128
// neighbouring bins 213 us), and the entries of a bracket crowd into the bins next to its lower end: in bin order a few
// channels would take them all, as the pass over the gradient with CFs 10, 100 and 1000 showed.
__device__ __forceinline__ uint32_t bin_word(uint32_t b) { return ((b & 63u) << 5) | (b >> 6); }
static_assert(NBIN == 64 * 32, "bin_word");

// Random-k: priority of index i, a keyed bijection of the 31-bit integers (adding a constant, multiplying
// by an odd constant and xor with a right shift are all bijections of [0, 2^31)), so no two indices tie.
__device__ __forceinline__ uint32_t priority_of(uint32_t s0, uint32_t s1, uint32_t i)
{
    const uint32_t M = 0x7FFFFFFFu;
    uint32_t x = (i + s0) & M;
    x ^= x >> 16; x = (x * 0x7FEB352Du) & M;
    x ^= x >> 15; x = (x * 0x046CA68Bu) & M;
    x ^= x >> 16; x = (x + s1) & M;
    x ^= x >> 14; x = (x * 0x2C1B3C6Du) & M;
    x ^= x >> 15; x = (x * 0x297A2D39u) & M;
    x ^= x >> 15;
    return x;
}

// The ordering key of a candidate: from its value (Top-k) or from its index (Random-k).
__device__ __forceinline__ uint32_t cand_key(const Params& p, int32_t idx, float val)
{
    return p.random ? priority_of(p.rk_s0, p.rk_s1, (uint32_t)idx) : key_of(val);
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Cross-lane sums with DPP (data-parallel primitives of the vector ALU) instead of LDS permutes: a step costs an
// instruction, not a round trip through the LDS crossbar, which matters where a wavefront's reductions sit on the
// critical path of a short kernel.  A row is 16 lanes; a lane whose source does not exist reads 0.
constexpr int DPP_QUAD_1032 = 0xB1, DPP_QUAD_2301 = 0x4E;       // quad_perm:[1,0,3,2], quad_perm:[2,3,0,1]
constexpr int DPP_ROW_SHR = 0x110, DPP_ROW_ROR = 0x120;         // + n: row_shr:n, row_ror:n
constexpr int DPP_ROW_BCAST15 = 0x142, DPP_ROW_BCAST31 = 0x143; // lane 15 of a row to the next row; lane 31 to rows 2 and 3

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true);
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ double dpp_move(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_move<CTRL, ROW_MASK>((uint32_t)b), hi = dpp_move<CTRL, ROW_MASK>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));   // a missing source gives +0.0
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint64_t dpp_move(uint64_t v)
{
    const uint32_t lo = dpp_move<CTRL, ROW_MASK>((uint32_t)v), hi = dpp_move<CTRL, ROW_MASK>((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ uint64_t last_lane(uint64_t v)
{
    return ((uint64_t)last_lane((uint32_t)(v >> 32)) << 32) | last_lane((uint32_t)v);
}
__device__ __forceinline__ double last_lane(double v)
{
    return __longlong_as_double((long long)last_lane((uint64_t)__double_as_longlong(v)));
}

// Sum over the 64 lanes, the same value (and for floating point the same order of additions) in every lane:
// pairs, quads, the row's four quads, then rows 0+1 and 2+3, then all in lane 63, which is broadcast.
template <typename T>
__device__ __forceinline__ T wave_sum_t(T v)
{
    v += dpp_move<DPP_QUAD_1032>(v);
    v += dpp_move<DPP_QUAD_2301>(v);
    v += dpp_move<DPP_ROW_ROR + 4>(v);
    v += dpp_move<DPP_ROW_ROR + 8>(v);
    v += dpp_move<DPP_ROW_BCAST15, 0xA>(v);
    v += dpp_move<DPP_ROW_BCAST31, 0xC>(v);
    return last_lane(v);
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return wave_sum_t(v); }
__device__ __forceinline__ double wave_sum(double v) { return wave_sum_t(v); }
__device__ __forceinline__ uint64_t wave_sum(uint64_t v) { return wave_sum_t(v); }

__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, dpp_move<DPP_QUAD_1032>(v));   // (the values are not negative: a missing source's +0.0 changes nothing)
    v = fmax(v, dpp_move<DPP_QUAD_2301>(v));
    v = fmax(v, dpp_move<DPP_ROW_ROR + 4>(v));
    v = fmax(v, dpp_move<DPP_ROW_ROR + 8>(v));
    v = fmax(v, dpp_move<DPP_ROW_BCAST15, 0xA>(v));
    v = fmax(v, dpp_move<DPP_ROW_BCAST31, 0xC>(v));
    return last_lane(v);
}

// inclusive prefix sum over the lanes of a wavefront: within the rows first, then the earlier rows' totals
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    uint32_t s = v + dpp_move<DPP_ROW_SHR + 1>(v);
    s += dpp_move<DPP_ROW_SHR + 2>(v);
    s += dpp_move<DPP_ROW_SHR + 3>(v);
    s += dpp_move<DPP_ROW_SHR + 4>(s);
    s += dpp_move<DPP_ROW_SHR + 8>(s);
    s += dpp_move<DPP_ROW_BCAST15, 0xA>(s);
    s += dpp_move<DPP_ROW_BCAST31, 0xC>(s);
    return s;
}

__device__ __forceinline__ uint32_t hash32(uint32_t x)
{
    x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
    return x;
}

// v[0] out, the others one place down: a rolled loop over registers.  The list kernels are short chains that start with
// a cold instruction cache, and unrolled copies of their long bodies (50 KB) cost them more than the moves.
template <typename T, int N>
__device__ __forceinline__ T pop_front(T (&v)[N])
{
    const T x = v[0];
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) v[i] = v[i + 1];
    return x;
}

// A sub-tile's word in brk_cnt: entries in its bracket list, and the number of zeros that were counted instead of listed.
constexpr uint32_t ZERO_SHIFT = 16, LISTED = (1u << ZERO_SHIFT) - 1u;
static_assert(TS <= (int)LISTED, "both fit");

// What a wavefront of the list kernels works on, a unit: the U sub-tiles from U u on, U = SUB (a tile) or, in calls of few
// tiles, MIDDLE or FINE (units_per_tile).  The entries of a unit's lists are the concatenation of
// its sub-tile lists.
template <int U>
struct UnitLists {
    uint32_t start[U + 1];  // start[j] = entries in sub-tiles before j; start[U] = all
    uint32_t zeros;         // the bracket lists: zeros that are not in them
    __device__ __forceinline__ uint32_t total() const { return start[U]; }
    // slot (relative to the unit's first slot) of the unit's i-th entry
    __device__ __forceinline__ uint32_t slot(uint32_t i) const
    {
        uint32_t j = 0;
#pragma unroll
        for (int x = 1; x < U; ++x) j += (i >= start[x]);
        uint32_t s = 0;
#pragma unroll
        for (int x = 1; x < U; ++x) if ((uint32_t)x == j) s = start[x];
        return j * TS + (i - s);
    }
};

// the bracket lists
template <int U>
__device__ __forceinline__ UnitLists<U> bracket_lists(const Params& p, uint32_t u)
{
    UnitLists<U> c;
    c.start[0] = 0;
    c.zeros = 0;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const uint32_t x = p.brk_cnt[(size_t)u * U + j];
        c.start[j + 1] = c.start[j] + (x & LISTED);
        c.zeros += x >> ZERO_SHIFT;
    }
    return c;
}

// Four wavefronts (threads q = 0..255 of a 256-thread team; `q` is the thread's number inside the team, `scratch` 8
// words of LDS owned by the team) search a 2048-bin histogram for the bin of the k-th largest: thread q holds the
// counts h of bins 8q .. 8q+7, and the first wavefront's `extra` are more counts of the last bin.  Scanning from the top
// bin down, above < k <= above + count; every thread gets the result, bin == NONE if there are fewer than k entries.
// The caller provides the barrier: `sync()` must cover at least the team.
template <typename Sync>
__device__ __forceinline__ void team_locate_bin(uint32_t h[8], uint32_t extra, uint32_t k, int q, uint32_t* scratch, Sync sync,
                                                uint32_t& bin, uint32_t& above, uint32_t& count)
{
    const int lane = q & 63, wv = q >> 6;
    extra = wave_sum(extra);  // non-zero in the team's first wavefront only
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) mine += h[i];
    const uint32_t incl = wave_scan(mine);
    if (lane == 63) scratch[wv] = incl;
    if (q == 0) scratch[4] = extra;
    sync();
    const uint32_t ex = scratch[4];  // belongs to the very last bin
    uint32_t total = ex, before = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        total += scratch[x];
        if (x < wv) before += scratch[x];
    }
    uint32_t ab = total - ex - (before + incl);  // entries in the bins above this thread's eight ...
    if (q == 255) h[7] += ex;
    else ab += ex;                               // ... including the extra counts of the last bin
    uint32_t fb = NONE, fa = 0, fc = 0;
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        if (ab < k && ab + h[i] >= k) { fb = 8 * q + i; fa = ab; fc = h[i]; }
        ab += h[i];
    }
    sync();  // scratch is rewritten below
    if (fb != NONE) { scratch[5] = fb; scratch[6] = fa; scratch[7] = fc; }
    if (q == 0) scratch[4] = (total >= k) ? 1u : 0u;
    sync();
    if (scratch[4]) { bin = scratch[5]; above = scratch[6]; count = scratch[7]; }
    else { bin = NONE; above = 0; count = 0; }
    sync();
}

// ---------------------------------------------------------------------------------------------
// S: layerwise mode, a tensor of at most SMALL_MAX elements: ONE workgroup does the whole step for it
// (error feedback, exact selection for every CF, statistics, message, residual) out of LDS, with no
// sample, no histogram in memory and no tile bookkeeping.  Its place in the message is known on the
// host (k_t is a function of the tensor's size), so nothing waits for it.  Runs as extra workgroups of
// the threshold kernel's launch (the workgroups that would otherwise have nothing to do for such a tensor).
// ---------------------------------------------------------------------------------------------
constexpr int SMALL_MAX = TW;              // elements
constexpr int SM_T = 1024;                 // threads
constexpr int SM_W = SM_T / 64;
constexpr int SM_PER = SMALL_MAX / SM_T;   // consecutive elements per thread
static_assert(SM_PER == 8, "see small_at");

struct SmallShared {
    float a[SMALL_MAX + SMALL_MAX / 32];   // acc, element i at i + i / 32: the runs of eight of 32 neighbouring threads
                                           // then fall into different banks
    uint32_t hist[256];
    uint32_t wg[SM_W], we[SM_W];
    uint32_t pick[2];
    uint32_t tau[MAXCF], need[MAXCF];      // per CF, kept by thread 0 for the statistics
    double ds[MAXCF + 1][SM_W];
};

__device__ __forceinline__ int small_at(int i) { return i + (i >> 5); }

__device__ __forceinline__ void small_segment(const Params& p, int t, SmallShared& sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    const int64_t s0 = p.segs[t].begin;
    const int nt = (int)(p.segs[t].end - s0);
    const int64_t koff = p.segs[t].koff;
    // acc into LDS, coalesced: all loads first and without branches around them (an element past the end reads the
    // last one instead and is not stored), so that they are in flight together
    {
        float gv[SM_PER], rv[SM_PER];
#pragma unroll
        for (int q = 0; q < SM_PER; ++q) {
            const int i = q * SM_T + tid;
            gv[q] = p.grad[s0 + (i < nt ? i : nt - 1)];
            rv[q] = 0.0f;
        }
        if (!p.single) {
#pragma unroll
            for (int q = 0; q < SM_PER; ++q) {
                const int i = q * SM_T + tid;
                rv[q] = p.res[s0 + (i < nt ? i : nt - 1)];
            }
        }
#pragma unroll
        for (int q = 0; q < SM_PER; ++q) {
            const int i = q * SM_T + tid;
            if (i < nt) sh.a[small_at(i)] = p.single ? gv[q] : rv[q] + gv[q];
        }
    }
    __syncthreads();
    // this thread's run: elements SM_PER tid .. SM_PER tid + nv - 1
    const int first = SM_PER * tid;
    const int nv = nt - first < 0 ? 0 : (nt - first > SM_PER ? SM_PER : nt - first);
    // (the keys stay in registers; the values are read from LDS again where they are needed)
    uint32_t key[SM_PER];
    double ssd = 0.0;
#pragma unroll
    for (int e = 0; e < SM_PER; ++e) {
        const float v = e < nv ? sh.a[small_at(first + e)] : 0.0f;
        key[e] = p.random ? priority_of(p.rk_s0, p.rk_s1, (uint32_t)(s0 + first + e)) : key_of(v);
        const double d = (double)v;
        ssd += d * d;
    }
    {
        const double w = wave_sum(ssd);
        if (lane == 0) sh.ds[MAXCF][wib] = w;
    }
    uint32_t tau_c = 0, need_c = 0;
    for (int j = 0; j < p.n_cf; ++j) {
        // the k-th largest key by four passes over the key's digits (8, 8, 8 and 7 bits from the top), each a
        // 256-bin histogram of the keys that agree with the digits found so far
        uint32_t want = p.ktab[(size_t)t * p.n_cf + j];
        uint32_t prefix = 0, mask = 0;
#pragma unroll 1
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = pass == 0 ? 23 : pass == 1 ? 15 : pass == 2 ? 7 : 0;
            const uint32_t dm = pass == 3 ? 127u : 255u;
            if (tid < 256) sh.hist[tid] = 0;
            __syncthreads();
            // (magnitudes crowd into a few digit values: a thread adds runs of equal digits at once)
            uint32_t cur = NONE, run = 0;
#pragma unroll
            for (int e = 0; e < SM_PER; ++e) {
                if (e < nv && (key[e] & mask) == prefix) {
                    const uint32_t dg = (key[e] >> shift) & dm;
                    if (dg != cur) {
                        if (run) atomicAdd(&sh.hist[cur], run);
                        cur = dg; run = 0;
                    }
                    ++run;
                }
            }
            if (run) atomicAdd(&sh.hist[cur], run);
            __syncthreads();
            if (wib == 0) {
                // lane l owns digits 4 l .. 4 l + 3; from the top: above < want <= above + count
                const uint32_t h0 = sh.hist[4 * lane], h1 = sh.hist[4 * lane + 1], h2 = sh.hist[4 * lane + 2], h3 = sh.hist[4 * lane + 3];
                const uint32_t mine = h0 + h1 + h2 + h3;
                const uint32_t incl = wave_scan(mine);
                const uint32_t total = __shfl(incl, 63, 64);
                uint32_t ab = total - incl;
                const uint32_t hh[4] = {h0, h1, h2, h3};
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    if (ab < want && ab + hh[q] >= want) { sh.pick[0] = 4u * lane + q; sh.pick[1] = ab; }
                    ab += hh[q];
                }
            }
            __syncthreads();
            prefix |= sh.pick[0] << shift;
            mask |= dm << shift;
            want -= sh.pick[1];
        }
        if (tid == 0) { sh.tau[j] = prefix; sh.need[j] = want; }   // want: the keys equal to tau that are selected
        if (j == p.commit) { tau_c = prefix; need_c = want; }
        // energy above the threshold (Random-k: and of the entry at it, which has no particular magnitude)
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < SM_PER; ++e) {
            if (e < nv && (key[e] > prefix || (p.random && key[e] == prefix))) {
                const double d = (double)sh.a[small_at(first + e)];
                s += d * d;
            }
        }
        s = wave_sum(s);
        if (lane == 0) sh.ds[j][wib] = s;
    }
    // the committed CF's selection, in index order: a thread's run is consecutive, so the counts of the threads
    // before it give its place
    uint32_t g = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < SM_PER; ++e) {
        g += (e < nv && key[e] > tau_c);
        eq += (e < nv && key[e] == tau_c);
    }
    const uint32_t ig = wave_scan(g), ie = wave_scan(eq);
    if (lane == 63) { sh.wg[wib] = ig; sh.we[wib] = ie; }
    __syncthreads();
    uint32_t run_g = ig - g, run_e = ie - eq;
#pragma unroll
    for (int w = 0; w < SM_W; ++w)
        if (w < wib) { run_g += sh.wg[w]; run_e += sh.we[w]; }
    const uint32_t ties_before = run_e < need_c ? run_e : need_c;
    int64_t o = koff + run_g + ties_before;
    const int64_t lim = koff + (int64_t)p.ktab[(size_t)t * p.n_cf + p.commit];
    uint32_t left = need_c - ties_before;
#pragma unroll
    for (int e = 0; e < SM_PER; ++e) {
        if (e >= nv) continue;
        bool sel = key[e] > tau_c;
        if (key[e] == tau_c && left > 0) { sel = true; --left; }
        if (sel) {
            if (o < lim) {   // (always, if the counts are consistent; never write out of range)
                p.out_val[o] = sh.a[small_at(first + e)];
                p.out_idx[o] = p.single ? p.map_idx[s0 + first + e] : (int32_t)(s0 + first + e);
            }
            ++o;
            if (!p.no_commit) sh.a[small_at(first + e)] = 0.0f;
        }
    }
    if (tid == 0) {
        // statistics: every wavefront's sums in order
        double ss_dense = 0.0;
        for (int w = 0; w < SM_W; ++w) ss_dense += sh.ds[MAXCF][w];
        for (int j = 0; j < p.n_cf; ++j) {
            double s = 0.0;
            for (int w = 0; w < SM_W; ++w) s += sh.ds[j][w];
            const double tauv = p.random ? (double)sh.tau[j] : (double)__uint_as_float(sh.tau[j]);
            if (!p.random) s += (double)sh.need[j] * tauv * tauv;
            double* os = p.out_stats + ((size_t)t * p.n_cf + j) * GRAVAC_STATS_PER_CF;
            os[0] = s;
            os[1] = ss_dense;
            os[2] = (ss_dense == 0.0) ? 1.0 : s / ss_dense;
            os[3] = tauv;
        }
    }
    __syncthreads();
    // the new residual (acc with the selection zeroed), coalesced; single-source mode: into the dense residual
#pragma unroll 4
    for (int q = 0; q < SM_PER; ++q) {
        const int i = q * SM_T + tid;
        if (i >= nt) continue;
        const float r = sh.a[small_at(i)];
        if (!p.single) {
            p.res[s0 + i] = r;
        } else if (p.restore) {
            const int mi = p.map_idx[s0 + i];
            if ((uint64_t)(int64_t)mi < (uint64_t)p.n_restore) p.restore[mi] = r;
        }
    }
}

// A call's status record and, where the host knows it, the number of pairs: by one workgroup of its first kernel that has
// something to do for every call of its kind.
__device__ __forceinline__ void reset_status(const Params& p, uint32_t tid)
{
    if (tid != 0) return;
    p.status->any_fail = 0; p.status->n_fail = 0; p.status->error = 0; p.status->n_seg = p.n_seg;
    p.status->n_narrow = 0; p.status->count = 0; p.status->n_wide = 0;
    if (p.out_count && p.bounds_from != BOUNDS_FIXED) *p.out_count = p.total_out;  // (else the last step knows it)
}

// The bracket of CF j of segment t where no sample is needed: it follows from k alone (Random-k) or is left empty (every
// segment takes the exact route).  w: lo, hi, mid.
__device__ __forceinline__ void known_bracket(const Params& p, int t, int j, uint32_t* w)
{
    uint32_t lo = NONE, hi = NONE, mid = NONE;
    if (p.bounds_from == BOUNDS_RANDOM) {
        // priorities are a keyed permutation of the 31-bit integers: the number of a tensor's nt indices
        // with priority >= x is as good as binomial (nt, 1 - x / 2^31), so the bounds follow from k alone:
        // x with k + ZMARGIN sqrt(k) + 2 expected above it, and x with k - ZMARGIN sqrt(k) - 2
        const uint64_t nt = (uint64_t)(seg_end(p, t) - seg_begin(p, t));
        const double k = (double)seg_k(p, t, j), w0 = ZMARGIN * sqrt(k) + 2.0;
        const double q_lo = (k + w0) / (double)nt, q_hi = (k - w0) / (double)nt;
        lo = q_lo >= 1.0 ? 0u : (uint32_t)floor(2147483648.0 * (1.0 - q_lo));
        hi = q_hi <= 0.0 ? KEY_END : (uint32_t)ceil(2147483648.0 * (1.0 - q_hi));
        mid = (uint32_t)floor(2147483648.0 * (1.0 - (k >= (double)nt ? 1.0 : k / (double)nt)));
    }
    w[0] = lo; w[1] = hi; w[2] = mid;
}

// Ranks in the sample, S of nt elements, whose keys are a bracket's ends and the estimate of the k-th largest.
__device__ __forceinline__ void sampled_ranks(uint32_t k, uint32_t S, uint64_t nt, uint32_t& r_lo, uint32_t& r_hi, uint32_t& r_mid)
{
    r_lo = r_hi = r_mid = k;
    if ((uint64_t)S == nt) return;   // the whole segment was read
    // expected number of sampled keys among the k largest, widened by ZMARGIN standard deviations
    const double m = (double)k * (double)S / (double)nt, sd = sqrt(m);
    const double a = ceil(m + ZMARGIN * sd + 2.0), b = floor(m - ZMARGIN * sd - 2.0);
    r_lo = (a >= 4.0e9) ? NONE : (uint32_t)a;
    r_hi = (b < 1.0) ? 1u : (uint32_t)b;
    r_mid = (m < 1.0) ? 1u : (m >= 4.0e9 ? NONE : (uint32_t)(m + 0.5));
}

// The r_mid-th sample from the top is the (r_mid - above)-th of the c in sample bin `bin`: that far down from the bin's upper
// edge, as if the bin's samples were spread evenly over its keys.
__device__ __forceinline__ uint32_t key_inside(uint32_t bin, uint32_t w0, uint32_t down_of, uint32_t c)
{
    const uint32_t first = sample_bin_first(bin, w0), end = sample_bin_end(bin, w0);
    // (an estimate: single precision will do, and keeps a 64-bit division out of the kernel)
    const uint32_t down = (uint32_t)((float)(end - first) * ((float)down_of / (float)c));
    return down >= end - first ? first : end - down;
}

// ---------------------------------------------------------------------------------------------
// K0a: sample acc = residual + grad at stratified positions; each workgroup histograms its samples in
// LDS (SBIN bins, see sample_bin) and stores the counts as 16-bit numbers, and beside them how many of its
// samples lie above each of RGRP groups of bins.  The same launch clears what the later kernels
// add to (every workgroup a share of its segment's histograms and counters); a call whose brackets
// do not come from a sample launches it for that alone.
// ---------------------------------------------------------------------------------------------
template <int R>  // R groups per thread: a workgroup histograms R * SAMPLE_BLOCK samples
__global__ __launch_bounds__(256) void sample_kernel(Params p)
{
    __shared__ uint32_t h[SBIN];
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    const int t = is_flat(p) ? 0 : (int)p.sblock_seg[b];
    const uint32_t lb = b - (is_flat(p) ? 0u : p.segs[t].samp0);
    const uint32_t S = is_flat(p) ? p.flat_samples : p.segs[t].samp_cnt;
    const auto clear = [&]() {
        // the segment's sample blocks share the clearing: block lb of nbk takes every nbk-th 16-byte piece
        const uint32_t per = SAMPLE_BLOCK * R;
        const uint32_t nbk = is_flat(p) ? p.n_sample_blocks : (S + per - 1) / per;
        const uint4 z = make_uint4(0u, 0u, 0u, 0u);
        const uint32_t blocks = (uint32_t)p.n_cf * seg_rep(p, t);  // the segment's copy blocks
        for (uint32_t i = lb * 256 + tid; i < blocks; i += nbk * 256) p.list_cnt[(seg_block(p, t, 0) + i) * 32] = 0;
        if (is_flat(p) && b == 0) reset_status(p, tid);   // (a flat call has no threshold step)
        if (p.direct) return;
        if (lb == 0 && tid < XQ_WORDS) p.xq[(size_t)t * XQ_LINE + tid] = 0;
        uint4* h1 = (uint4*)(p.hist1 + seg_block(p, t, 0) * NBIN);
        for (uint32_t i = lb * 256 + tid; i < blocks * NBIN / 4; i += nbk * 256) h1[i] = z;
        uint4* cs = (uint4*)(p.coarse + (size_t)t * NBIN);
        for (uint32_t i = lb * 256 + tid; i < NBIN / 4; i += nbk * 256) cs[i] = z;
        for (uint32_t i = lb * 256 + tid; i < (uint32_t)p.n_cf * 64; i += nbk * 256) p.ovfc[((size_t)t * p.n_cf * 64 + i) * 32] = 0;
        if (is_flat(p) && b == 0 && p.bounds_from != BOUNDS_SAMPLED && tid < p.n_cf) known_bracket(p, 0, tid, p.bnd + 4 * tid);
        if (p.csum)
            for (uint32_t i = b * 256 + tid; i < p.n_csum; i += gridDim.x * 256) p.csum[(size_t)i * 8] = 0;
    };
    if (p.bounds_from != BOUNDS_SAMPLED) {
        clear();
        return;
    }
    const int64_t s0 = seg_begin(p, t);
    const uint64_t nt = (uint64_t)(seg_end(p, t) - s0);
    // The window: every block of the segment looks at the same 256 elements, 64 groups of four spread evenly, and takes the
    // exponent of the largest (an infinite or NaN one does not count).  Their loads are issued before the sample's and
    // arrive with them.  (256 single elements are four times the memory the sample itself takes: a call with 1000 tensors of
    // 20,000 elements spent 55 us here instead of 28, and all together 191 instead of 171.)
    const uint64_t wat = ((nt * (2u * (tid >> 2) + 1u)) >> 7) + (tid & 3u), wpos = wat < nt ? wat : nt - 1u;
    const float wg = p.grad[s0 + (int64_t)wpos], wr = p.single ? 0.0f : p.res[s0 + (int64_t)wpos];
    __shared__ uint32_t wexp[4];
    // A group is 4 consecutive elements: sample i of the segment is element i % 4 of group i / 4.  A sampled
    // segment (S a multiple of SAMPLE_BLOCK, nt > 2 S) is cut into S / 16 strata of at least 32 elements, and the
    // four groups of a stratum are the 16 elements of one line at a hashed place inside it: a sample costs a
    // sixteenth of the memory transactions that single elements at scattered places would (the sampling pass is
    // bound by their number, not by their bytes).
    static_assert(SAMPLE_BLOCK / 256 == 4, "groups of four");
    constexpr int Q = 4 * R;
    uint64_t gpos[R];
    bool live[Q];
    // stratum g of G = S / 16 spans [g step / 2^32, (g + 1) step / 2^32) with step = 2^32 nt / G, which is off by less than 2^10
    // and G less than 2^15: the last stratum ends at nt or just before.  (64-bit and 32-bit divisions for the exact ends and the
    // place inside took 1 us before the first load.)
    const uint32_t G = S / 16 ? S / 16 : 1u;
    static_assert(SAMPLE_MAX_FLAT / 16 <= 1 << 15, "g step fits 64 bits: nt < 2^31");
    const uint64_t step = (uint64_t)((double)nt * 4294967296.0 / (double)G);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t g = (lb * R + r) * (SAMPLE_BLOCK / 4) + tid;  // group
        gpos[r] = 4ull * g;                                          // the whole segment is read: elements 4g .. 4g+3
        if ((uint64_t)S != nt) {
            // four neighbouring threads share one stratum and one run of 16 elements in it that starts at a multiple
            // of 16 in the flat buffer (a 64-byte line if the buffer is aligned to that)
            const uint32_t g16 = g >> 2;
            const uint64_t a = (g16 * step) >> 32, e = ((g16 + 1u) * step) >> 32;     // e - a >= 32 (nt > 32 G), e <= nt
            const uint64_t first = ((uint64_t)s0 + a + 15) & ~15ull;                 // first such run inside the stratum
            const uint32_t runs = (uint32_t)(((uint64_t)s0 + e - first) / 16);        // >= 1
            const uint64_t at = first + 16ull * __umulhi(hash32(g16 * 0x9E3779B9u + 0x85EBCA6Bu), runs);
            gpos[r] = (at - (uint64_t)s0) + 4u * (g & 3u);                            // gpos + 3 < e <= nt
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) live[4 * r + q] = 4ull * g + q < S;
    }
    // all loads first, without branches around them (a group past the segment's last sample reads the segment's
    // last element instead and is not counted), so that they are in flight together
    float gv[Q], rv[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint64_t pos = gpos[q / 4] + (q & 3) < nt ? gpos[q / 4] + (q & 3) : nt - 1;
        gv[q] = p.grad[s0 + (int64_t)pos];
        rv[q] = 0.0f;
    }
    if (!p.single) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint64_t pos = gpos[q / 4] + (q & 3) < nt ? gpos[q / 4] + (q & 3) : nt - 1;
            rv[q] = p.res[s0 + (int64_t)pos];
        }
    }
    // while they are on their way
    clear();
#pragma unroll
    for (int q = 0; q < SBIN / 256; ++q) h[q * 256 + tid] = 0;
    const uint32_t wk = key_of(p.single ? wg : wr + wg);
    const double m = wave_max(wk < 0x7F800000u ? (double)(wk >> 23) : 0.0);
    if ((tid & 63) == 0) wexp[tid >> 6] = (uint32_t)m;
    __syncthreads();   // (... and the histogram is cleared)
    uint32_t e = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) e = wexp[w] > e ? wexp[w] : e;
    // exponents e + SWIN_ABOVE + 1 - SWIN .. e + SWIN_ABOVE, inside the octaves covered
    // (not the lowest: the first bin holds the keys below them, too)
    uint32_t b0 = e + SWIN_ABOVE + 1u > SWIN + SEXP0 + 1u ? e + SWIN_ABOVE + 1u - SWIN : SEXP0 + 1u;
    b0 = b0 > SEXP0 + SOCT - SWIN ? SEXP0 + SOCT - SWIN : b0;
    const uint32_t w0 = b0 << 23;
    if (lb == 0 && tid == 0) p.xq[(size_t)t * XQ_LINE + XQ_WIN] = w0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const float acc = p.single ? gv[q] : rv[q] + gv[q];
        if (live[q]) atomicAdd(&h[sample_bin(key_of(acc), w0)], 1u);
    }
    __syncthreads();
    // thread i stores bins 16i .. 16i+15, two counts per word (a count is at most R * SAMPLE_BLOCK < 2^16)
    static_assert(R * SAMPLE_BLOCK < 65536, "16-bit counts");
    uint4 w[2];
    uint32_t* wp = (uint32_t*)w;
    uint32_t mine = 0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const uint32_t c0 = h[16 * tid + 2 * m], c1 = h[16 * tid + 2 * m + 1];
        wp[m] = c0 | (c1 << 16);
        mine += c0 + c1;
    }
    uint4* dst = (uint4*)(p.samp_hist + (size_t)b * (SBIN / 2) + 8 * tid);
    dst[0] = w[0];
    dst[1] = w[1];
    // what lies above each group of SBIN / RGRP = 64 bins, four neighbouring threads' (a block's samples fit 16 bits)
    static_assert(SBIN / RGRP == 4 * 16, "four threads per group");
    const uint32_t incl = wave_scan(mine);
    if ((tid & 63) == 63) wexp[tid >> 6] = incl;   // (read before the last barrier)
    __syncthreads();
    uint32_t above = last_lane(incl) - incl;
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) above += w > (tid >> 6) ? wexp[w] : 0u;
    if ((tid & 3) == 3) p.samp_above[(size_t)b * RGRP + (tid >> 2)] = (uint16_t)above;
}

// ---------------------------------------------------------------------------------------------
// K0b: layerwise, per segment, add up the sample histograms and turn the sampled ranks into a bracket of keys per
// CF.  (Flat calls have bracket_kernel.)  G workgroups per segment; workgroup y adds up the bins [y, y + 1) * SBIN / G of all the
// segment's sample blocks (what lies above them it knows from the blocks' group counts) and writes the
// bracket ends that fall into its bins, so that no workgroup waits for another.  The kernels that
// use the brackets derive the histogram shift and the rest from them (bracket_bins).
// ---------------------------------------------------------------------------------------------
// (the form with the small tensors is held to 64 registers, so that two of its 1024-thread workgroups fit a CU: a
// layerwise call has more such workgroups than the chip has CUs)
template <int G, bool SMALL, int P = 1>  // SMALL: the workgroups of tensors of at most SMALL_MAX elements do the whole step for them
__global__ __launch_bounds__(P * 1024 / G) __attribute__((amdgpu_waves_per_eu(SMALL ? 8 : 1, 8))) void threshold_kernel(Params p)
{
    constexpr int T = 1024 / G;          // thread i < T owns the bins 4 (y T + i) .. + 3: two words of every block's histogram
    // P threads per such set of bins: thread i + x T adds up the blocks x, x + P, ..., of which a tensor has up to 64: one round
    // of loads per thread with P = 2, two with P = 1 (tensors of 30 million, 20,000 and 1 million elements 109.4 us with one, 106.5
    // with two, 105.5 with four threads; twenty of 2 million 129.3, 128.9 and 128.8; thirty of 65,537 45.1, 45.7 and 44.5)
    static_assert(P * 1024 / G <= 1024 && (G > 1 || P == 1), "threads of a workgroup");
    constexpr int NW = T / 64;
    static_assert(G == 1 || G == SGRP, "one workgroup per group of bins, or one for all");
    __shared__ uint32_t wtot[NW], gab[NW];
    __shared__ uint32_t rank_lo[MAXCF], rank_hi[MAXCF], rank_mid[MAXCF];
    __shared__ uint32_t hx[P > 1 ? P - 1 : 1][P > 1 ? T : 1][4];
    const int t = blockIdx.x, y = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    const int part = tid / T, ot = tid - part * T;
    if (t == 0 && y == 0) reset_status(p, (uint32_t)tid);
    if constexpr (SMALL) {
        static_assert(G == 1 && SM_T == 1024, "the small tensors' workgroups are this kernel's");
        __shared__ SmallShared small;
        if (seg_small(p, t)) {
            small_segment(p, t, small);
            return;
        }
    }
    const uint32_t S = p.segs[t].samp_cnt;
    const uint32_t sb0 = p.segs[t].samp0;
    const uint32_t nb = (S + SAMPLE_BLOCK - 1) / SAMPLE_BLOCK;
    const uint64_t nt = (uint64_t)(seg_end(p, t) - seg_begin(p, t));
    uint32_t* bnd = p.bnd + (size_t)t * BND_WORDS;
    if (y == 0) {
        for (uint32_t u = seg_tile0(p, t) + tid; u < seg_tile1(p, t); u += T * P) p.tseg[u] = (uint32_t)t;
        if (p.wseg)
            for (uint32_t i = tid; i < p.segs[t].wgs; i += T * P) p.wseg[p.segs[t].wg0 + i] = (uint32_t)t;
    }
    if (p.bounds_from != BOUNDS_SAMPLED) {
        if (y == 0 && tid < p.n_cf) known_bracket(p, t, tid, bnd + 4 * tid);
        return;
    }
    if (tid < p.n_cf) sampled_ranks(seg_k(p, t, tid), S, nt, rank_lo[tid], rank_hi[tid], rank_mid[tid]);
    // samples in the groups of bins above this workgroup's (fetched first and added up after the histograms)
    const uint32_t w0 = p.xq[(size_t)t * XQ_LINE + XQ_WIN];
    uint32_t g_above = 0;
    static_assert(G == 1 || 1024 / G >= SAMPLE_MAX_SEG * 2 / SAMPLE_BLOCK, "a block's count per thread covers a tensor's sample");
    if (G > 1 && part == 0 && (uint32_t)ot < nb) g_above = p.samp_above[(size_t)(sb0 + ot) * RGRP + (y + 1) * (RGRP / SGRP) - 1];
    uint32_t h0 = 0, h1 = 0, h2 = 0, h3 = 0;
    {
        const uint2* src = (const uint2*)(p.samp_hist + (size_t)sb0 * (SBIN / 2)) + (y * T + ot);
        constexpr int NB = SMALL ? 16 : 32;   // loads in flight per thread
        for (uint32_t b0 = (uint32_t)part; b0 < nb; b0 += NB * P) {
            uint2 w[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q) w[q] = (b0 + q * P < nb) ? src[(size_t)(b0 + q * P) * (SBIN / 4)] : make_uint2(0u, 0u);
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                h0 += w[q].x & 0xFFFFu; h1 += w[q].x >> 16;
                h2 += w[q].y & 0xFFFFu; h3 += w[q].y >> 16;
            }
        }
    }
    if (P > 1) {
        if (part != 0) {
            uint32_t* d = hx[part - 1][ot];
            d[0] = h0; d[1] = h1; d[2] = h2; d[3] = h3;
            h0 = h1 = h2 = h3 = 0;
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int x = 0; x < P - 1; ++x) { h0 += hx[x][ot][0]; h1 += hx[x][ot][1]; h2 += hx[x][ot][2]; h3 += hx[x][ot][3]; }
        }
    }
    if (G > 1 && part == 0) {
        g_above = wave_sum(g_above);
        if (lane == 0) gab[wib] = g_above;
    }
    const uint32_t mine = h0 + h1 + h2 + h3;
    const uint32_t incl = wave_scan(mine);
    if (lane == 63 && part == 0) wtot[wib] = incl;
    __syncthreads();
    if (part != 0) return;   // (no barrier follows)
    uint32_t local = 0, before = 0;
    g_above = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint32_t x = wtot[w];
        local += x;
        if (w < wib) before += x;
        if (G > 1) g_above += gab[w];
    }
    const uint32_t above0 = g_above + local - (before + incl);  // samples in bins above this thread's four
    const uint32_t hh[4] = {h0, h1, h2, h3};
    for (int j = 0; j < p.n_cf; ++j) {
        const uint32_t r_lo = rank_lo[j], r_hi = rank_hi[j], r_mid = rank_mid[j];
        uint32_t above = above0;
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            const uint32_t c = hh[q];
            const uint32_t bin = 4u * (uint32_t)(y * T + ot) + (uint32_t)q;
            // lower edge of the bin of the r_lo-th sample from the top, upper edge of the bin of the r_hi-th
            if (above < r_lo && above + c >= r_lo) bnd[4 * j] = sample_bin_first(bin, w0);
            if (above < r_hi && above + c >= r_hi) bnd[4 * j + 1] = sample_bin_end(bin, w0);
            if (above < r_mid && above + c >= r_mid) bnd[4 * j + 2] = key_inside(bin, w0, r_mid - above, c);
            above += c;
        }
        // fewer samples than a rank: the bracket is open on that side
        if (y == 0 && tid == 0) {
            if (S < r_lo) bnd[4 * j] = 0u;
            if (S < r_hi) bnd[4 * j + 1] = KEY_END;
            if (S < r_mid) bnd[4 * j + 2] = NONE;
        }
    }
}

// From which key on the pass over the gradient stores +0 instead of acc in a sub-tile that lists its candidates
// (NONE: nowhere): the key the sample puts the committed CF's k-th largest at, kept inside that CF's bracket
// [lo, top).  Entries from there on are in the candidate list, and most of them are selected: the emit step then has
// a scattered store only for the entries between this key and the threshold, selected ones below it (+0) or
// unselected ones at or above it (acc put back), instead of one for every selected entry of the bracket; a
// scattered 4-byte store costs the memory a read and a write of its 64 bytes, 34 us per million of them.
__device__ __forceinline__ uint32_t zero_from(const Params& p, uint32_t lo, uint32_t top, uint32_t mid)  // mid: bnd_mid
{
    if (p.single || p.no_commit || top == KEY_END) return NONE;
    if (mid == NONE) return top;
    return mid < lo ? lo : (mid > top ? top : mid);
}

// A flat call's brackets: RGRP wavefronts, each of which adds up one group of bins of all sample blocks' histograms (what
// lies above them it knows from the blocks themselves) and writes the bracket ends that fall into its bins.  No wavefront
// waits for another, and up to 64 blocks are one round trip to memory.
// (As a part of the pass, whose other wavefronts waited for it with their loads on their way, it was no faster: under the
// pass's own traffic the round trips take two to three times as long.  25 MB buckets 64 -> 66 us, the ResNet101 shape 123.4
// -> 121.7 at CF 100 and 164 -> 167 with three CFs.)
template <bool D>  // a direct call
__global__ __launch_bounds__(64) void bracket_kernel(Params p)
{
    const uint32_t role = blockIdx.x, nb = p.n_sample_blocks, S = p.flat_samples;
    const int lane = threadIdx.x;
    // (one round trip for up to 64 blocks: what lies above the group in block `lane`, two bins of every second block)
    const uint32_t w0 = p.xq[XQ_WIN], k = p.flat_k[lane < p.n_cf ? lane : 0];
    uint32_t g_above = 0;
    for (uint32_t b = lane; b < nb; b += 64) g_above += p.samp_above[b * RGRP + role];
    static_assert(SBIN / RGRP == 64 && RGRP == 64, "half a wavefront covers a group's words, two bins each");
    const uint32_t half = (uint32_t)lane >> 5;
    const uint32_t* src = p.samp_hist + (size_t)role * 32u + (lane & 31);
    uint32_t h0 = 0, h1 = 0;
    constexpr uint32_t NB = 32;   // loads in flight
#pragma unroll 1
    for (uint32_t b0 = 0; b0 < nb; b0 += 2 * NB) {
        uint32_t w[NB];
#pragma unroll
        for (uint32_t q = 0; q < NB; ++q) {
            const uint32_t b = b0 + 2 * q + half;
            w[q] = src[(b < nb ? b : nb - 1u) * (SBIN / 2)];
        }
#pragma unroll
        for (uint32_t q = 0; q < NB; ++q)
            if (b0 + 2 * q + half < nb) { h0 += w[q] & 0xFFFFu; h1 += w[q] >> 16; }
    }
    uint32_t rank_lo, rank_hi, rank_mid;
    sampled_ranks(k, S, (uint64_t)p.n, rank_lo, rank_hi, rank_mid);
    h0 += __shfl_xor(h0, 32, 64);
    h1 += __shfl_xor(h1, 32, 64);
    if (half != 0u) h0 = h1 = 0;
    g_above = wave_sum(g_above);
    const uint32_t incl = wave_scan(h0 + h1);
    const uint32_t above1 = g_above + last_lane(incl) - incl, above0 = above1 + h1;   // samples above each of this lane's bins
    const uint32_t bin0 = 2u * (role * 32u + (uint32_t)(lane & 31));
    for (int j = 0; j < p.n_cf; ++j) {
        if constexpr (D) {
            // all ranks are k, and all elements are counted: the bin of the k-th largest and what lies above it
            const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)rank_lo, j);
            const bool in1 = above1 < kj && above1 + h1 >= kj, in0 = above0 < kj && above0 + h0 >= kj;
            if (__ballot(in1 || in0) == 0ull) continue;
            const uint32_t bin = in1 ? bin0 + 1u : bin0, above = in1 ? above1 : above0, c = in1 ? h1 : h0;
            // (the first and the last bin span many octaves, too many for sums scaled by the bin's bounds)
            const uint32_t width = sample_bin_end(bin, w0) - sample_bin_first(bin, w0);
            const bool wide = width != 1u && (c > (uint32_t)LCAP || width > (1u << SCSHIFT));
            if (__ballot((in1 || in0) && wide) != 0ull) {
                // where the emit step counts it again, and its queue
                if (lane < XQ_WORDS) p.xq[lane] = 0;
                uint4* h = (uint4*)wide_hist(p, j, 0);
                for (uint32_t i = lane; i < WIDE_ROUNDS * NBIN / 4; i += 64) h[i] = make_uint4(0u, 0u, 0u, 0u);
            }
            if (in1 || in0) {
                const uint32_t lo = sample_bin_first(bin, w0), end = sample_bin_end(bin, w0), mid = key_inside(bin, w0, kj - above, c);
                CfState st;
                st.k = kj; st.lo = lo; st.s = 0; st.base = lo; st.span = end - lo - 1u; st.above = above; st.c = c; st.top = end;
                st.mode = st.span == 0u ? MODE_RESOLVED : wide ? MODE_WIDE : MODE_GATHER;
                st.tau = lo; st.cnt_gt = above; st.need = kj - above;   // (if resolved)
                st.pad[0] = st.pad[1] = st.pad[2] = st.pad[3] = 0;
                p.st[j] = st;
                p.bnd[4 * j] = lo; p.bnd[4 * j + 1] = end; p.bnd[4 * j + 2] = mid; p.bnd[4 * j + 3] = st.mode;
                if (wide) { p.status->any_fail = 1; p.status->n_fail = 1; p.status->n_narrow = 1; p.status->n_wide = 1; }
                if (j == p.commit) {
                    SegState sg;
                    sg.fail = FAIL_NONE; sg.pz = zero_from(p, lo, end, mid);
                    p.seg[0] = sg;
                }
            }
        } else {
            const auto find = [&](uint32_t ranks, uint32_t word, uint32_t none, auto key) {
                // the bin of the rank-th sample from the top, if it is one of this wavefront's
                const uint32_t rank = (uint32_t)__builtin_amdgcn_readlane((int)ranks, j);
                const bool in1 = above1 < rank && above1 + h1 >= rank, in0 = above0 < rank && above0 + h0 >= rank;
                const uint64_t m = __ballot(in1 || in0);
                if (m != 0ull) {
                    const uint32_t value = key(in1 ? bin0 + 1u : bin0, rank - (in1 ? above1 : above0), in1 ? h1 : h0);
                    if (in1 || in0) p.bnd[4 * j + word] = value;
                } else if (role == 0u && S < rank) {
                    if (lane == 0) p.bnd[4 * j + word] = none;   // fewer samples than a rank: the bracket is open on that side
                }
            };
            // lower edge of the bin of the rank_lo-th sample from the top, upper edge of the bin of the rank_hi-th
            find(rank_lo, 0u, 0u, [&](uint32_t bin, uint32_t, uint32_t) { return sample_bin_first(bin, w0); });
            find(rank_hi, 1u, KEY_END, [&](uint32_t bin, uint32_t, uint32_t) { return sample_bin_end(bin, w0); });
            find(rank_mid, 2u, NONE, [&](uint32_t bin, uint32_t down, uint32_t c) { return key_inside(bin, w0, down, c); });
        }
    }
}

// ---------------------------------------------------------------------------------------------
// K1: the pass over the gradient, one sub-tile per wavefront.
//     SM_EF: read grad and residual, write acc back, sum acc^2.
//     SM_EXACT (exact route, failed segments only): read acc from residual; the brackets come from the
//     coarse histogram.  Both collect the lists of the sub-tile in index order.
// ---------------------------------------------------------------------------------------------
// Entries of a sub-tile that some bracket concerns (key >= lo_min) go through LDS on their way to the lists, compacted in
// index order, so that what has to be done for each of them (per CF a count and an energy, a histogram update; the list
// stores) is done 64 entries at a time by full wavefronts.  Done where the entries lie, an element at a time, the pass
// over the ResNet101 shape with CFs 10, 100 and 1000 took 800 vector instructions and 61 stores and atomics per sub-tile, a
// few lanes each, and 120 us instead of 106 (the LSTM shape with two CFs 107 -> 103 us).  16 KB per workgroup leave the occupancy to the registers.
constexpr uint32_t STAGE = 512;   // entries a wavefront can hold
static_assert(STAGE >= 2 * ROW && DENSE_SUB <= STAGE, "a row fits behind another, and a sub-tile with a candidate list in one piece");

template <int NCF>  // compiled for calls with up to NCF CFs: the loops over the CFs are unrolled
struct SubCtx {
    uint32_t lo_min, lo_c, pz;
    uint32_t lo[NCF];
    uint32_t org[NCF];
    uint32_t sh[NCF];
    uint32_t top[NCF];
    uint32_t ovn[NCF];     // entries above CF j's bracket (the same in all lanes) ...
    double ovs[NCF];       // ... and their sum of acc^2 (this lane's share)
    uint32_t* h1;   // this wavefront's copy of the bracket histograms of the tile's segment ...
    uint32_t hstride;  // ... whose CFs are this many words apart
    int32_t* cidx;  // candidate-list slots of this sub-tile
    float* cval;
    uint32_t run;   // candidates listed so far
    uint32_t* bkey; // bracket-list slots of this sub-tile
    float* bval;
    uint32_t brun;  // bracket entries listed so far
    double ssd;
    int ncf;
    uint32_t s0, s1;  // Random-k keys
    uint2* stage;     // this wavefront's entries in LDS: index and value ...
    uint32_t staged;  // ... and their number
    uint32_t wide;    // a direct call: bit j: the entries of CF j's bin are not gathered (MODE_WIDE)
};

__device__ __forceinline__ v4f ld_stream(const v4fu* q)
{
#if GV_NT
    return __builtin_nontemporal_load(q);
#else
    return *q;
#endif
}

__device__ __forceinline__ void st_stream(v4f v, v4fu* q)
{
#if GV_NT
    __builtin_nontemporal_store(v, q);
#else
    *q = v;
#endif
}

// The ordering keys of one lane's four consecutive elements a[0..3] at global index g.
template <bool RND, int NCF>
__device__ __forceinline__ void keys_of_row(const SubCtx<NCF>& c, const float a[4], int64_t g, uint32_t key[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) key[e] = RND ? priority_of(c.s0, c.s1, (uint32_t)(g + e)) : key_of(a[e]);
}

// One lane's four consecutive elements a[0..3] with keys key[0..3] at global index g; vm = validity bits: those that some
// bracket concerns are staged behind what is there (index order: lanes, then a lane's elements).
template <int NCF>
__device__ __forceinline__ void stage_row(SubCtx<NCF>& c, const float a[4], const uint32_t key[4], int64_t g, unsigned vm)
{
    bool f[4];
    uint64_t m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[e] = ((vm >> e) & 1u) && key[e] >= c.lo_min;
        m[e] = __ballot(f[e]);
    }
    if ((m[0] | m[1] | m[2] | m[3]) == 0ull) return;
    uint32_t w = c.staged;
#pragma unroll
    for (int e = 0; e < 4; ++e) w += lanes_below(m[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (f[e]) {
            c.stage[w] = make_uint2((uint32_t)(g + e), __float_as_uint(a[e]));
            ++w;
        }
        c.staged += (uint32_t)__popcll(m[e]);
    }
}

// The same for a row of a sub-tile that keeps no candidate list.  Most of its entries lie above the bracket, which is all
// there is to know of them: they are counted here, and only those inside it are staged (the VGG16 shape at CF 10, whose
// convolutions are such sub-tiles: 397 -> 394 us).  For one CF: with more, the code costs every call registers (three CFs on
// the ResNet101 shape 164 -> 168 us), and all entries are staged.
__device__ __forceinline__ void stage_dense_row(SubCtx<1>& c, const float a[4], const uint32_t key[4], int64_t g)
{
    unsigned in = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double d = (double)a[e], dd = d * d;
        const bool from = key[e] >= c.lo_min, above = from && key[e] >= c.top[0];
        c.ovn[0] += (uint32_t)__popcll(__ballot(above));
        c.ovs[0] += above ? dd : 0.0;
        in |= (from && !above) ? 1u << e : 0u;
    }
    stage_row<1>(c, a, key, g, in);
}

// The staged entries, 64 at a time: per CF a count and the energy of those above its bracket and a histogram update for
// those inside it; into the lists.  listed = whether the sub-tile keeps a candidate list; counted = whether the entries above
// the bracket have been counted.
// D (a direct call): those inside a bracket go to the gather lists, unless they are too many; zeros are counted where they are
// found.
template <bool RND, bool D, int NCF>
__device__ __forceinline__ void flush_stage(const Params& p, uint32_t v, SubCtx<NCF>& c, bool listed, bool counted, int lane)
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the wavefront's own LDS writes, read back by other lanes
#pragma unroll 1
    for (uint32_t b = 0; b < c.staged; b += 64) {
        const bool live = b + lane < c.staged;
        const uint2 s = c.stage[b + lane];   // (b + lane < STAGE, a multiple of 64)
        const float val = __uint_as_float(s.y);
        const uint32_t key = RND ? priority_of(c.s0, c.s1, s.x) : key_of(val);
        const double d = (double)val, dd = d * d;
        bool inside = false;
#pragma unroll
        for (int j = 0; j < NCF; ++j) {
            if (j == 0 || j < c.ncf) {
                const bool from = live && key >= c.lo[j], above = from && key >= c.top[j];
                if (!counted) {
                    c.ovn[j] += (uint32_t)__popcll(__ballot(above));
                    c.ovs[j] += above ? dd : 0.0;
                }
                const bool in = from && !above && !(D && key == 0u);
                const uint64_t m = __ballot(in);
                if (m == 0ull) continue;
                if (D && ((c.wide >> j) & 1u)) {
                    // (the bracket list has them)
                } else if constexpr (D) {
                    const uint32_t lst = (uint32_t)j * REP + (blockIdx.x & (REP - 1u));
                    const int leader = __ffsll((unsigned long long)m) - 1;
                    uint32_t at = 0;
                    if (lane == leader) at = atomicAdd(&p.list_cnt[lst * 32], (uint32_t)__popcll(m));
                    const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)at, leader) + lanes_below(m);
                    if (in && pos < LCAP) {
                        p.list_key[lst * LCAP + pos] = key;
                        p.list_tile[lst * LCAP + pos] = v / FINE;
                    }
                } else {
                    if (in) atomicAdd(&c.h1[j * c.hstride + bin_word((key - c.org[j]) >> c.sh[j])], 1u);
                }
                inside = inside || in;
            }
        }
        if (listed) {
            const bool cand = live && key >= c.lo_c;
            const uint64_t m = __ballot(cand);
            if (cand) {
                const uint32_t w = c.run + lanes_below(m);
                c.cidx[w] = (int32_t)s.x;
                c.cval[w] = val;
            }
            c.run += (uint32_t)__popcll(m);
        }
        const uint64_t m = __ballot(inside);
        if (inside) {
            const uint32_t w = c.brun + lanes_below(m);
            c.bkey[w] = key;
            if (RND) c.bval[w] = val;
        }
        c.brun += (uint32_t)__popcll(m);
    }
    c.staged = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // read before the next entries overwrite them
}

// Modes of the pass.
enum { SM_EF = 0,      // acc = residual + grad, written back into residual
       SM_EXACT = 1,   // exact route: acc is re-read, the lists are collected again
       SM_SINGLE = 2   // single source (second-level compression): acc = grad; every value is also written
};                     // back into the dense residual at its mapped index (the emit pass zeroes the selected)

// Issue the loads of one row (this lane's four elements from global index g).
template <int M>
__device__ __forceinline__ void row_load(const Params& p, int64_t g, v4f& x, v4f& y, v4i& m)
{
    if (M == SM_EF) { x = ld_stream((const v4fu*)(p.res + g)); y = ld_stream((const v4fu*)(p.grad + g)); }
    if (M == SM_EXACT) x = ld_stream((const v4fu*)(p.acc + g));
    if (M == SM_SINGLE) {
        y = ld_stream((const v4fu*)(p.grad + g));
        if (p.restore) m = *(const v4iu*)(p.map_idx + g);
    }
}

// Arithmetic of one row; a[] gets the four acc values.
template <int M>
__device__ __forceinline__ void row_finish(const Params& p, const v4f& x, const v4f& y, const v4i& m, float a[4])
{
    if (M == SM_EF) {
        const v4f av = x + y;  // stored once the keys are known
        a[0] = av.x; a[1] = av.y; a[2] = av.z; a[3] = av.w;
    }
    if (M == SM_EXACT) { a[0] = x.x; a[1] = x.y; a[2] = x.z; a[3] = x.w; }
    if (M == SM_SINGLE) {
        a[0] = y.x; a[1] = y.y; a[2] = y.z; a[3] = y.w;
        if (p.restore) {
            const int mi[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((uint64_t)(int64_t)mi[e] < (uint64_t)p.n_restore) p.restore[mi[e]] = a[e];
        }
    }
}

// One element of a ragged sub-tile's row.
template <int M>
__device__ __forceinline__ float element_load(const Params& p, int64_t q)
{
    if (M == SM_EF) return p.res[q] + p.grad[q];
    if (M == SM_EXACT) return p.acc[q];
    const float a = p.grad[q];
    if (p.restore) {
        const int mi = p.map_idx[q];
        if ((uint64_t)(int64_t)mi < (uint64_t)p.n_restore) p.restore[mi] = a;
    }
    return a;
}

// The brackets with which the exact route collects a segment's lists again (in LDS).
struct ExactBounds {
    uint32_t lo[MAXCF];
    uint32_t sh[MAXCF];
    uint32_t top[MAXCF];   // first key past the bracket
    uint32_t* hist;        // the histograms' first copy of CF 0; LCAP words between copies
};

// One sub-tile v, by one wavefront; stage: STAGE entries of LDS of its own.
template <int M, bool RND, bool D, int NCF>
__device__ __forceinline__ void stream_subtile(const Params& p, uint32_t v, int lane, const ExactBounds* xb, uint2* stage)
{
    constexpr bool EF = (M != SM_EXACT);  // a first pass: sums acc^2, takes the brackets that were sampled
    const uint32_t u = v / SUB;  // tile
    if (u >= p.n_tiles) return;
    const int t = tile_seg(p, u);
    const int64_t sb = seg_begin(p, t), se = seg_end(p, t);
    const int64_t s0 = sb + (int64_t)(u - seg_tile0(p, t)) * TW + (int64_t)(v % SUB) * TS;
    const int64_t e0 = (s0 + TS < se) ? s0 + TS : se;
    const bool whole = e0 - s0 == TS;
    const uint32_t rep = seg_rep(p, t);
    const size_t block0 = seg_block(p, t, 0);
    // the brackets' load, then all rows': on their way together
    uint32_t word = NONE;   // lane 4 j + i: word i of CF j's bracket
    if (EF) {
        if (p.bounds_from == BOUNDS_FIXED) word = (lane & 3) == 2 ? NONE : p.fixed_key;   // an empty bracket at the caller's threshold
        else word = p.bnd[(size_t)t * BND_WORDS + (lane & (BND_WORDS - 1))];
    }
    float a[ROWS][4];
    if (whole) {
        v4f x[ROWS], y[ROWS];
        v4i mi[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) row_load<M>(p, s0 + q * ROW + 4 * lane, x[q], y[q], mi[q]);
#pragma unroll
        for (int q = 0; q < ROWS; ++q) row_finish<M>(p, x[q], y[q], mi[q], a[q]);
    }
    if (s0 >= se) {  // sub-tile past the end of the segment
        if (lane == 0) { p.cand_cnt[v] = 0; p.brk_cnt[v] = 0; if (EF) p.ssd[v] = 0.0; }
        if (lane < p.n_cf) { p.ovn[(size_t)v * p.n_cf + lane] = 0; p.ovs[(size_t)v * p.n_cf + lane] = 0.0; }
        return;
    }

    SubCtx<NCF> c;
    c.ncf = p.n_cf;
    c.s0 = p.rk_s0; c.s1 = p.rk_s1;
    c.lo_min = NONE; c.lo_c = NONE; c.pz = NONE; c.wide = 0;
#pragma unroll
    for (int j = 0; j < NCF; ++j) {
        c.ovn[j] = 0; c.ovs[j] = 0.0;
        c.lo[j] = NONE; c.org[j] = NONE; c.sh[j] = 0; c.top[j] = KEY_END;
    }
    if (EF) {
#pragma unroll
        for (int j = 0; j < NCF; ++j) {
            if (j < p.n_cf) {
                c.lo[j] = (uint32_t)__builtin_amdgcn_readlane((int)word, 4 * j);
                bracket_bins(c.lo[j], (uint32_t)__builtin_amdgcn_readlane((int)word, 4 * j + 1), c.sh[j], c.org[j], c.top[j]);
                c.lo_min = c.lo[j] < c.lo_min ? c.lo[j] : c.lo_min;
                if (D) {
                    c.top[j] = (uint32_t)__builtin_amdgcn_readlane((int)word, 4 * j + 1);   // (the bin, no more)
                    c.wide |= (uint32_t)__builtin_amdgcn_readlane((int)word, 4 * j + 3) == MODE_WIDE ? 1u << j : 0u;
                }
                if (j == p.commit) {
                    c.lo_c = c.lo[j];
                    if (M == SM_EF) c.pz = zero_from(p, c.lo[j], c.top[j], (uint32_t)__builtin_amdgcn_readlane((int)word, 4 * j + 2));
                }
            }
        }
    } else {
        static_assert(EF || NCF == MAXCF, "the exact route is compiled for any number of CFs");
#pragma unroll
        for (int j = 0; j < NCF; ++j) {
            if (j < p.n_cf) {
                c.lo[j] = c.org[j] = xb->lo[j]; c.sh[j] = xb->sh[j]; c.top[j] = xb->top[j];
                c.lo_min = c.lo[j] < c.lo_min ? c.lo[j] : c.lo_min;
                if (j == p.commit) c.lo_c = c.lo[j];
            }
        }
    }
    // the copy of the histogram this wavefront adds to, spread by the sub-tile number
    c.hstride = rep * (EF ? NBIN : LCAP);
    if (EF) c.h1 = p.hist1 + (block0 + ((v ^ (v / SUB)) & (rep - 1u))) * NBIN;
    else c.h1 = xb->hist + ((v ^ (v / SUB)) & (rep - 1u)) * LCAP;
    c.cidx = p.cand_idx + (size_t)v * TS;
    c.cval = p.cand_val + (size_t)v * TS;
    c.bkey = p.brk_key + (size_t)v * TS;
    c.bval = p.brk_val + (size_t)v * TS;
    c.run = 0;
    c.brun = 0;
    c.ssd = 0.0;
    c.stage = stage;
    c.staged = 0;

    bool dense = false;
    uint32_t rk[RND ? ROWS : 1][4];  // Random-k: the priorities, each computed once (four quarter-rate multiplications)
    bool at_once = false;            // all rows are staged before the entries are worked on
    // Zeros inside a bracket are only counted, not listed (whole sub-tiles of Top-k's first pass).  Where they may be
    // selected, the committed CF's bracket starts at zero, all of the sub-tile are candidates and it keeps no list.
    const bool count_zeros = EF && !RND && c.lo_min == 0u, skip_zeros = count_zeros && whole;
    if (skip_zeros) c.lo_min = 1u;
    uint32_t zeros = 0;
    int parts = (int)((e0 - s0 + ROW - 1) / ROW);
    if (whole) {
        uint32_t nc = 0, nm = 0;  // candidates for the message in this sub-tile, entries that some bracket concerns
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
            uint32_t key[4];
            keys_of_row<RND, NCF>(c, a[q], s0 + q * ROW + 4 * lane, key);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (RND) rk[q][e] = key[e];
                nm += (uint32_t)__popcll(__ballot(key[e] >= c.lo_min));
                if (NCF > 1) nc += (uint32_t)__popcll(__ballot(key[e] >= c.lo_c));
                if (EF) {
                    const double d = (double)a[q][e];   // (the square is exact in binary64: rounded once, as a sum of its own)
                    c.ssd = __builtin_fma(d, d, c.ssd);
                }
            }
        }
        zeros = skip_zeros ? (uint32_t)TS - nm : 0u;
        if (NCF == 1) nc = nm + zeros;
        dense = nc >= DENSE_SUB;
        if (M == SM_EF) {
            // acc goes back into the residual; in a sub-tile that keeps a candidate list an entry above the committed
            // CF's bracket leaves +0 there already: it is selected unless the bracket fails (the list keeps its value,
            // and the exact route puts it back), which spares the emit step a scattered store per selected entry
            const uint32_t z = dense ? NONE : c.pz;   // (a key is less than NONE)
#pragma unroll
            for (int q = 0; q < ROWS; ++q) {
                uint32_t key[4];
                if (RND) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) key[e] = rk[q][e];
                } else {
                    keys_of_row<RND, NCF>(c, a[q], 0, key);
                }
                v4f o;
                o.x = key[0] >= z ? 0.0f : a[q][0];
                o.y = key[1] >= z ? 0.0f : a[q][1];
                o.z = key[2] >= z ? 0.0f : a[q][2];
                o.w = key[3] >= z ? 0.0f : a[q][3];
                st_stream(o, (v4fu*)(p.res + s0 + q * ROW + 4 * lane));
            }
        }
        at_once = nm <= STAGE && !(NCF == 1 && dense);
        parts = nm == 0u ? 0 : (at_once ? 1 : ROWS);
    }
#pragma unroll 1
    for (int part = 0; part < parts; ++part) {
        if (at_once) {
#pragma unroll
            for (int q = 0; q < ROWS; ++q) {
                uint32_t key[4];
                if (RND) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) key[e] = rk[q][e];
                } else {
                    keys_of_row<RND, NCF>(c, a[q], 0, key);
                }
                stage_row<NCF>(c, a[q], key, s0 + q * ROW + 4 * lane, 0xFu);
            }
        } else {
            // a row at a time: one of many entries' rows, or the next of a ragged sub-tile, element-wise, guarded
            const int64_t g = s0 + part * ROW + 4 * lane;
            unsigned vm = whole ? 0xFu : 0u;
            if (!whole) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t q = g + e;
                    a[0][e] = 0.0f;
                    if (q < e0) {
                        vm |= 1u << e;
                        a[0][e] = element_load<M>(p, q);
                    }
                }
            }
            uint32_t key[4];
            keys_of_row<RND, NCF>(c, a[0], g, key);
            if (!whole) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (!((vm >> e) & 1u)) continue;
                    if (M == SM_EF) p.res[g + e] = key[e] >= c.pz ? 0.0f : a[0][e];
                    if (EF) {
                        const double d = (double)a[0][e];
                        c.ssd = __builtin_fma(d, d, c.ssd);
                    }
                }
                if (D && count_zeros) {   // (they are listed as candidates, if they are, but not as the bracket's)
#pragma unroll
                    for (int e = 0; e < 4; ++e) zeros += (uint32_t)__popcll(__ballot(((vm >> e) & 1u) && key[e] == 0u));
                }
            }
            if constexpr (NCF == 1) {
                if (dense) stage_dense_row(c, a[0], key, g);
                else stage_row<NCF>(c, a[0], key, g, vm);
            } else {
                stage_row<NCF>(c, a[0], key, g, vm);
            }
#pragma unroll
            for (int q = 0; q + 1 < ROWS; ++q) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[q][e] = a[q + 1][e];
            }
        }
        if (part == parts - 1 || c.staged > STAGE - ROW) flush_stage<RND, D, NCF>(p, v, c, !dense, NCF == 1 && dense, lane);
    }

#pragma unroll
    for (int j = 0; j < NCF; ++j) {
        if (j < p.n_cf) {
            const uint32_t o = c.ovn[j];
            const double s = wave_sum(c.ovs[j]);
            if (lane == 0) {
                p.ovn[(size_t)v * p.n_cf + j] = o;
                p.ovs[(size_t)v * p.n_cf + j] = s;
                if (EF && !D && o) atomicAdd(&p.ovfc[(((size_t)t * p.n_cf + j) * 64 + (v & 63)) * 32], o);
            }
        }
    }
    if (EF) {
        const double s = wave_sum(c.ssd);
        if (lane == 0) p.ssd[v] = s;
    }
    if (!D && zeros != 0u && lane == 0) {
#pragma unroll
        for (int j = 0; j < NCF; ++j)   // (a sampled bracket is not empty: zeros are inside one that starts there)
            if (c.lo[j] == 0u) atomicAdd(&c.h1[j * c.hstride + bin_word(0u)], zeros);
    }
    if (lane == 0) { p.cand_cnt[v] = dense ? DENSE_BIT : c.run; p.brk_cnt[v] = c.brun | (zeros << ZERO_SHIFT); }
}

// The first pass (SM_EF, SM_SINGLE): one sub-tile per wavefront, one launch covers the whole gradient.
template <int M, bool RND, bool D, int NCF>
__global__ __launch_bounds__(WG) void stream_kernel(Params p)
{
    static_assert(M != SM_EXACT, "the exact route is part of the plan step");
    __shared__ uint2 stage[WAVES][STAGE];
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * WAVES + (threadIdx.x >> 6));
    stream_subtile<M, RND, D, NCF>(p, w, threadIdx.x & 63, nullptr, stage[threadIdx.x >> 6]);
    if (p.bounds_from == BOUNDS_FIXED) {
        // the threshold sparsifier's first kernel.  The later steps find everything resolved: selected <=> key > tau with tau
        // one key below the threshold, no ties to take
        const uint32_t i = blockIdx.x * WG + threadIdx.x;
        if (p.csum && i < p.n_csum) p.csum[(size_t)i * 8] = 0;
        if (i == 0) {
            reset_status(p, 0);
            CfState st;
            st.k = 0; st.lo = p.fixed_key; st.s = 0; st.mode = MODE_RESOLVED; st.base = p.fixed_key; st.span = 0;
            st.above = 0; st.c = 0; st.tau = p.fixed_key - 1u; st.need = 0; st.cnt_gt = 0;
            st.top = p.fixed_key; st.pad[0] = st.pad[1] = st.pad[2] = st.pad[3] = 0;
            p.st[0] = st;
            SegState sg;
            sg.fail = FAIL_NONE; sg.pz = p.single ? NONE : p.fixed_key;
            p.seg[0] = sg;
        }
    }
}

// The candidates of sub-tile v that its first pass replaced by +0 in the residual get their values back (the
// sub-tile's candidate list holds them; nobody else touches the sub-tile).  By one wavefront.
__device__ __forceinline__ void put_back_subtile(const Params& p, uint32_t v, uint32_t pz, int lane)
{
    const uint32_t cc = p.cand_cnt[v];
    if (cc & DENSE_BIT) return;  // such a sub-tile kept acc
    const float* cv = p.cand_val + (size_t)v * TS;
    const int32_t* ci = p.cand_idx + (size_t)v * TS;
    for (uint32_t i0 = 0; i0 < cc; i0 += 64 * 4) {
        float vq[4];
        int32_t iq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t i = i0 + q * 64 + lane;
            vq[q] = cv[i < cc ? i : 0u];
            iq[q] = ci[i < cc ? i : 0u];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (i0 + q * 64 + lane < cc && cand_key(p, iq[q], vq[q]) >= pz) p.res[iq[q]] = vq[q];
    }
}

// How the bin that holds the k-th largest gets resolved to one key.
struct BinPlan {
    uint32_t mode, base, bits, above, c;   // (the bin spans 2^bits keys)
};

// Decide from the located bin (b, above, c) of the bracket histogram with bins (key - org) >> s; what lies above the
// bracket arrives as bin OVF.
__device__ __forceinline__ BinPlan plan_bin(uint32_t lo, uint32_t org, uint32_t s, uint32_t b, uint32_t above, uint32_t c)
{
    BinPlan q;
    const bool zero = lo == 0u && b == 0u;          // the bin of the key 0
    if (b == NONE || b == OVF) q.mode = MODE_FAIL;  // fewer than k entries from lo on, or the k-th lies above the bracket
    else if (s == 0 || zero) q.mode = MODE_RESOLVED;
    else if (c <= LCAP) q.mode = MODE_GATHER;
    else q.mode = MODE_FAIL;
    q.base = (b == NONE || b == OVF || zero) ? 0u : org + (b << s);
    q.bits = zero ? 0u : s;
    q.above = above;
    q.c = c;
    return q;
}

// ---------------------------------------------------------------------------------------------
// PLAN: find the bracket-histogram bin of every CF's k-th largest and decide how to resolve it.  All workgroups of a
//       segment (all of the launch in flat mode) work that out for themselves, which costs a few redundant reads of the
//       histograms and spares a kernel boundary: a segment whose bracket has not failed is done with that, and the
//       workgroups of one whose bracket has go on with the exact route in the same launch, without anybody having had to
//       tell them.  (As three launches, the locate step and two that found nothing to do, a call took 2 to 3 us more: on
//       the ResNet101 shape at CF 100 132.9 -> 129.9 us, 1 MiB buckets 40.1 -> 38.3 us.  The exact routes themselves, forced
//       on that shape: 474 -> 397 us with one CF, 780 -> 517 us with three; a mass of equal values, which the last step
//       used to count again alone, 357 -> 40 ms.)
//
// Exact routes.  The segment's tiles are cut into chunks, which the running workgroups claim from a counter; a
// workgroup keeps its chunks through all phases, so that what one phase writes for a tile (residual, lists) is read by
// the same workgroup in the next, and only histograms, made of device-wide atomics, pass between workgroups.  A
// workgroup waits for the others only when every chunk has been claimed, that is, for workgroups that are running and do
// not wait for anybody before they have finished the phase: the wait ends whatever else shares the chip and however few
// of this launch's workgroups are resident.  (Two calls at a time on one workspace break that; the wait is bounded for them.)
//   FAIL_FULL: phase 0 puts back what the pass replaced by +0 in the residual and histograms key >> 20 of all elements;
//              phase 1 collects the lists again with the located 2^20 keys as bracket, in bins of 2^9 keys.
//   FAIL_NARROW, FAIL_TIES: the located bin is cut into up to NBIN parts and counted again from the bracket lists.
//   Phase 2:   a bin that is still too full is cut again, which leaves bins one key wide (22 = 11 + 11 bits at most).
// ---------------------------------------------------------------------------------------------
constexpr int PLAN_T = 1024;            // threads: four teams that search one CF's histogram each
constexpr int PLAN_W = PLAN_T / 64;
constexpr uint32_t PLAN_GRID = 256;     // workgroups of a flat call, one per CU
constexpr uint32_t PLAN_HELP = 64;      // layerwise: tiles of a large tensor per further workgroup
constexpr uint32_t PLAN_CHUNKS = 4096;  // chunks of a segment at most
constexpr int CSUB = 8;  // copies of the coarse histogram inside a workgroup: lane l counts in copy l % CSUB
constexpr int XSHIFT = 9;               // bins of 2^XSHIFT keys cover the 2^20 keys of a coarse bin
static_assert((NBIN << XSHIFT) == (1 << 20) && LCAP == 2 * NBIN && XQ_WORDS >= 4, "two histograms per gather list; a counter per phase");

struct PlanShared {
    ExactBounds xb;
    uint32_t scratch[PLAN_T / 256][8];
    uint32_t fb[MAXCF], fa[MAXCF], fc[MAXCF];   // what the search found: bin, entries above it, entries in it
    uint32_t k[MAXCF], lo[MAXCF], s[MAXCF], top[MAXCF];
    uint32_t mode[MAXCF], base[MAXCF], above[MAXCF], c[MAXCF];
    uint32_t bs[MAXCF];                         // the located bin spans 2^bs keys
    uint32_t cut[MAXCF];                        // 1: it is being cut again, into parts of 2^s2 keys
    uint32_t s2[MAXCF];
    uint32_t pz;                                // SegState::pz
    uint32_t got, n_own, leader, arrived;
    uint32_t own[PLAN_CHUNKS];                  // the chunks this workgroup has claimed
    // Gradient magnitudes crowd into a few exponents, so most lanes of a wavefront hit the same few bins and LDS atomics
    // on one copy serialise 64-fold; CSUB copies cut that to 64 / CSUB.  (a row is one word longer than the histogram,
    // so that the CSUB counters of one bin lie in different banks)
    // (once they are counted: the wavefronts' staged entries while the lists are collected again)
    __attribute__((aligned(16))) uint32_t lh[CSUB][NBIN + 1];
};
static_assert(sizeof(uint32_t) * CSUB * (NBIN + 1) >= sizeof(uint2) * STAGE * PLAN_W, "the staged entries fit into the coarse counts' LDS");

// All CFs' searches; setup(j, hist, copies, stride, extra, want) says what to search for CF j: a 2048-bin histogram (bin b
// at bin_word(b)) in `copies` arrays `stride` words apart that are added up (16-byte aligned), and 64 more counts for the last bin, one per
// cache line, or null.  Results in sh.fb / fa / fc.  Called by the whole workgroup.
// The step is one workgroup's reads (64 KB per CF of a large tensor) and a short chain of barriers behind them, so the
// reads of a call with one or two CFs are split over all four teams, which then add up through LDS.
template <typename Setup>
__device__ __forceinline__ void plan_search(PlanShared& sh, int n_cf, int tid, Setup setup)
{
    const int team = tid >> 8, q = tid & 255;
    const int subs = n_cf == 1 ? 4 : n_cf == 2 ? 2 : 1, at_once = 4 / subs;   // teams per CF, CFs per round
    const int sub = team % subs;
    uint32_t* part = &sh.lh[0][0];   // (the coarse counts are not in use while a search runs)
    for (int j0 = 0; j0 < n_cf; j0 += at_once) {
        const int jt = j0 + team / subs, j = jt < n_cf ? jt : n_cf - 1;
        const uint32_t *hist, *extra_at;
        uint32_t copies, stride, want, b, above, c;
        setup(j, hist, copies, stride, extra_at, want);
        uint32_t h[8], extra = (extra_at && sub == 0 && q < 64) ? extra_at[q * 32] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) h[i] = 0;
        const auto add = [&](const uint4 (&v)[2]) {
            h[0] += v[0].x; h[1] += v[0].y; h[2] += v[0].z; h[3] += v[0].w;
            h[4] += v[1].x; h[5] += v[1].y; h[6] += v[1].z; h[7] += v[1].w;
        };
        const auto fetch = [&](uint32_t r, uint4 (&v)[2]) {
            const uint4* hv = (const uint4*)(hist + (size_t)r * stride + 8 * q);
            v[0] = hv[0]; v[1] = hv[1];
        };
        if (jt < n_cf) {
            if (copies == (uint32_t)REP && subs == 4) {
                uint4 v[REP / 4][2];
#pragma unroll
                for (int r = 0; r < REP / 4; ++r) fetch(sub + 4 * r, v[r]);
#pragma unroll
                for (int r = 0; r < REP / 4; ++r) add(v[r]);
            } else if (copies == (uint32_t)REP && subs == 2) {
                uint4 v[REP / 2][2];
#pragma unroll
                for (int r = 0; r < REP / 2; ++r) fetch(sub + 2 * r, v[r]);
#pragma unroll
                for (int r = 0; r < REP / 2; ++r) add(v[r]);
            } else if (copies == (uint32_t)REP) {
                uint4 v[REP][2];
#pragma unroll
                for (int r = 0; r < REP; ++r) fetch(r, v[r]);
#pragma unroll
                for (int r = 0; r < REP; ++r) add(v[r]);
            } else {
                for (uint32_t r = sub; r < copies; r += subs) {
                    uint4 v[2];
                    fetch(r, v);
                    add(v);
                }
            }
        }
        // the words 8 q .. 8 q + 7 (bin_word order) go through LDS, which puts them into bin order and adds the teams up
#pragma unroll
        for (int i = 0; i < 8; ++i) part[(team * 8 + i) * 257 + q] = h[i];
        __syncthreads();
        if (sub == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t w = bin_word(8u * (uint32_t)q + (uint32_t)i);
                h[i] = part[(team * 8 + (w & 7u)) * 257 + (w >> 3)];
                for (int x = 1; x < subs; ++x) h[i] += part[((team + x) * 8 + (w & 7u)) * 257 + (w >> 3)];
            }
        }
        team_locate_bin(h, extra, want, q, sh.scratch[team], [] { __syncthreads(); }, b, above, c);
        if (q == 0 && sub == 0 && jt < n_cf) { sh.fb[j] = b; sh.fa[j] = above; sh.fc[j] = c; }
    }
    __syncthreads();
}
static_assert(4 * 8 * 257 <= CSUB * (NBIN + 1), "the teams' counts fit into the coarse counts' LDS");

// Everything this workgroup has written is visible to the device; then all workgroups with chunks of the segment have
// got here (the counter has grown to `target` by what each of them adds, the number of its chunks), and what they have written
// is visible to this one.  False (to every thread): they have not, after as many
// polls as the call allows.  That takes a second call on the same workspace, which clears this one's counters or claims
// its chunks; the wait must not hold the GPU for ever then.
__device__ __forceinline__ bool wait_for_all(const Params& p, uint32_t n_own, uint32_t& arrived, uint32_t* done, uint32_t target, int tid)
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // every wavefront's stores and atomics are done ...
    __syncthreads();
    if (tid == 0) {
        __threadfence();                                           // ... and leave this XCD's L2
        atomicAdd(done, n_own);
        uint32_t polls = 0;
        while (polls < p.wait_polls &&
               __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target + p.wait_extra) {
            __builtin_amdgcn_s_sleep(4);
            ++polls;
        }
        arrived = polls < p.wait_polls ? 1u : 0u;
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return arrived != 0u;
}

// One tile's entries of the bracket lists into the histograms (first copy of CF 0 at hist) of the CFs that are cut again.
__device__ __forceinline__ void plan_recount(const Params& p, const PlanShared& sh, uint32_t u, uint32_t* hist, uint32_t copies, int lane)
{
    const UnitLists<SUB> tl = bracket_lists<SUB>(p, u);
    const uint32_t cnt = tl.total();
    for (uint32_t i0 = 0; i0 < cnt; i0 += 64 * 8) {
        uint32_t kq[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t i = i0 + q * 64 + lane;
            kq[q] = p.brk_key[(size_t)u * TW + tl.slot(i < cnt ? i : 0u)];
        }
        for (int j = 0; j < p.n_cf; ++j) {
            if (!sh.cut[j]) continue;
            uint32_t* h = hist + ((size_t)j * copies + (u & (copies - 1u))) * LCAP;
            const uint32_t base = sh.base[j], top = sh.top[j], width = 1u << sh.bs[j], s2 = sh.s2[j];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                // (an entry counts if it lies inside the bracket the lists were collected with: what lies above was
                // counted as above the bracket by the pass and may be listed all the same)
                const bool in = i0 + q * 64 + lane < cnt && kq[q] < top && kq[q] >= base && kq[q] - base < width;
                const uint32_t bin = (kq[q] - base) >> s2;
                // a mass of equal keys: the lanes that share the first one's bin add once
                const uint64_t m = __ballot(in);
                if (m == 0ull) continue;
                const int first = __ffsll((unsigned long long)m) - 1;
                const uint64_t same = __ballot(in && bin == (uint32_t)__shfl((int)bin, first, 64));
                if (lane == first) atomicAdd(&h[bin_word(bin)], (uint32_t)__popcll(same));
                else if (in && !((same >> lane) & 1ull)) atomicAdd(&h[bin_word(bin)], 1u);
            }
        }
    }
}

template <bool RND>
__global__ __launch_bounds__(PLAN_T) void plan_kernel(Params p)
{
    __shared__ PlanShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    int t = 0;
    bool first_block = blockIdx.x == 0;   // of the segment
    if (!is_flat(p)) {
        if (blockIdx.x < (uint32_t)p.n_seg) {
            t = (int)blockIdx.x;
            first_block = true;
        } else {
            const uint32_t u = (blockIdx.x - (uint32_t)p.n_seg) * PLAN_HELP;
            if (u >= p.n_tiles) return;
            t = tile_seg(p, u);
            if (u - seg_tile0(p, t) < PLAN_HELP) return;   // (the segment's first workgroup is enough for these tiles)
            first_block = false;
        }
        if (seg_small(p, t)) return;
    }
    const uint32_t copies = seg_rep(p, t);
    const size_t id0 = (size_t)t * p.n_cf;
    // (the brackets are fetched along with the histograms)
    uint32_t b_lo = 0, b_hi = 0, b_mid = 0;
    if (tid < p.n_cf) { const uint32_t* b = p.bnd + (size_t)t * BND_WORDS + 4 * tid; b_lo = b[0]; b_hi = b[1]; b_mid = b[2]; }
    plan_search(sh, p.n_cf, tid, [&](int j, const uint32_t*& hist, uint32_t& nc, uint32_t& stride, const uint32_t*& extra, uint32_t& want) {
        hist = p.hist1 + seg_block(p, t, j) * NBIN; nc = copies; stride = NBIN;
        extra = p.ovfc + (id0 + j) * 64 * 32; want = seg_k(p, t, j);
    });
    if (tid < p.n_cf) {
        const int j = tid;
        const uint32_t lo = b_lo;
        uint32_t s, org, top;
        bracket_bins(lo, b_hi, s, org, top);
        if (j == p.commit) sh.pz = zero_from(p, lo, top, b_mid);
        const uint32_t b = sh.fb[j];
        const BinPlan q = plan_bin(lo, org, s, b, sh.fa[j], sh.fc[j]);
        sh.k[j] = seg_k(p, t, j); sh.lo[j] = lo; sh.s[j] = s; sh.top[j] = top;
        sh.mode[j] = q.mode; sh.base[j] = q.base; sh.above[j] = q.above; sh.c[j] = q.c; sh.bs[j] = q.bits;
    }
    __syncthreads();
    uint32_t kind = FAIL_NONE;
    for (int j = 0; j < p.n_cf; ++j) {
        if (sh.mode[j] != MODE_FAIL) continue;
        const uint32_t b = sh.fb[j];
        const uint32_t x = (b == NONE || b == OVF) ? FAIL_FULL : (sh.s[j] > 11u ? FAIL_NARROW : FAIL_TIES);
        kind = x > kind ? x : kind;
    }
    bool writes = first_block, counts = true;   // this workgroup records the plan, and counts the segment
    if (kind != FAIL_NONE) {
        // ---- exact routes
        uint32_t* xq = p.xq + (size_t)t * XQ_LINE;
        const uint32_t u0 = seg_tile0(p, t), u1 = seg_tile1(p, t), tiles = u1 - u0;
        // (two tiles are one sub-tile per wavefront; a few chunks per workgroup leave little of a last, uneven round)
        constexpr uint32_t UNIT = PLAN_W / SUB;
        const uint32_t per = UNIT * ((tiles + UNIT * PLAN_CHUNKS - 1) / (UNIT * PLAN_CHUNKS));  // tiles per chunk
        const uint32_t n_chunks = (tiles + per - 1) / per;
        uint32_t* xhist = p.list_key + seg_block(p, t, 0) * LCAP;   // the first of the two sets of histograms
        const bool full = kind == FAIL_FULL;
        const uint32_t pz = sh.pz;
        __syncthreads();   // (sh.lo / top / fb are rewritten below)
        if (tid == 0) { sh.n_own = 0; sh.leader = 0; }
        if (full)
            for (uint32_t i = tid; i < CSUB * (NBIN + 1); i += PLAN_T) (&sh.lh[0][0])[i] = 0;
        uint32_t next = tid == 0 ? atomicAdd(&xq[0], 1u) : 0u;
        for (;;) {
            if (tid == 0) sh.got = sh.n_own < PLAN_CHUNKS ? next : NONE;   // (more are not to be had, unless the counter was cleared)
            __syncthreads();
            const uint32_t at = sh.got;
            __syncthreads();
            if (at >= n_chunks) break;
            if (tid == 0) {
                sh.own[sh.n_own++] = at;
                if (at == 0) sh.leader = 1;
                next = atomicAdd(&xq[0], 1u);   // (on its way while this chunk is worked on)
            }
            if (at == 0) {
                const uint4 z = make_uint4(0u, 0u, 0u, 0u);
                uint4* h = (uint4*)xhist;
                for (uint32_t i = tid; i < (uint32_t)p.n_cf * copies * (LCAP / 4); i += PLAN_T) h[i] = z;
            }
            if (!full) continue;
            uint32_t* h = sh.lh[lane & (CSUB - 1)];
            const int64_t sb = seg_begin(p, t), se = seg_end(p, t);
            const uint32_t v1 = (u0 + (at + 1) * per < u1 ? u0 + (at + 1) * per : u1) * SUB;
            for (uint32_t v = (u0 + at * per) * SUB + wib; v < v1; v += PLAN_W) {
                const int64_t s0 = sb + (int64_t)(v - u0 * SUB) * TS;
                const int64_t e0 = (s0 + TS < se) ? s0 + TS : se;
                if (s0 >= se) continue;
                if (pz != NONE) {
                    // acc is read again from the residual: first put back what the first pass replaced by +0 there
                    put_back_subtile(p, v, pz, lane);
                    __threadfence_block();  // the loads below are this wavefront's own, of the same addresses
                }
                // all loads first, without branches around them (an element past the end reads the last one instead and
                // is not counted), so that they are in flight together
                static_assert(TS == 64 * 16, "a lane's loads cover the sub-tile");
                float a[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) a[r] = p.acc[s0 + lane + r * 64 < e0 ? s0 + lane + r * 64 : e0 - 1];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (s0 + lane + r * 64 < e0) atomicAdd(&h[cand_key(p, (int32_t)(s0 + lane + r * 64), a[r]) >> 20], 1u);
            }
        }
        if (sh.n_own == 0) return;   // every chunk is somebody else's
        writes = sh.leader != 0;
        if (full) {
            __syncthreads();
            uint32_t* gh = p.coarse + (size_t)t * NBIN;
            for (uint32_t i = tid; i < NBIN; i += PLAN_T) {
                uint32_t v = 0;
#pragma unroll
                for (int c = 0; c < CSUB; ++c) v += sh.lh[c][i];
                if (v) atomicAdd(&gh[bin_word(i)], v);
            }
        }
        bool arrived = wait_for_all(p, sh.n_own, sh.arrived, &xq[1], n_chunks, tid);
        if (full && arrived) {
            // the coarse (key >> 20) bin of every CF's k-th largest is the new bracket
            plan_search(sh, p.n_cf, tid, [&](int j, const uint32_t*& hist, uint32_t& nc, uint32_t& stride, const uint32_t*& extra, uint32_t& want) {
                hist = p.coarse + (size_t)t * NBIN; nc = 1; stride = NBIN; extra = nullptr; want = sh.k[j];
            });
            if (tid < p.n_cf) {
                uint32_t b = sh.fb[tid];
                if (b == NONE) { b = 0; p.status->error = 1; }
                sh.lo[tid] = b << 20; sh.s[tid] = XSHIFT; sh.top[tid] = (b + 1u) << 20;   // (2^31, KEY_END, at most)
                sh.above[tid] = sh.fa[tid]; sh.base[tid] = b << 20; sh.bs[tid] = 20; sh.s2[tid] = XSHIFT; sh.cut[tid] = 1;
                sh.xb.lo[tid] = b << 20; sh.xb.sh[tid] = XSHIFT; sh.xb.top[tid] = (b + 1u) << 20;
            }
        } else if (!full && tid < p.n_cf) {
            const bool x = sh.mode[tid] == MODE_FAIL;
            sh.cut[tid] = x ? 1u : 0u;
            sh.s2[tid] = sh.bs[tid] > 11u ? sh.bs[tid] - 11u : 0u;
        }
        if (tid == 0) sh.xb.hist = xhist;
        __syncthreads();
        for (int phase = 1; phase <= 2 && arrived; ++phase) {
            uint32_t* hist = xhist + (phase - 1) * NBIN;
            // the workgroup's chunks, dealt over its wavefronts by the sub-tile or by the tile
            const uint32_t per_chunk = full && phase == 1 ? per * SUB : per, all = sh.n_own * per_chunk;
            for (uint32_t i = wib; i < all; i += PLAN_W) {
                const uint32_t x = i / per_chunk, first = u0 + sh.own[x] * per;
                if (full && phase == 1) {
                    const uint32_t v = __builtin_amdgcn_readfirstlane(first * SUB + (i - x * per_chunk));
                    if (v < u1 * SUB) stream_subtile<SM_EXACT, RND, false, MAXCF>(p, v, lane, &sh.xb, (uint2*)&sh.lh[0][0] + wib * STAGE);
                } else {
                    const uint32_t u = first + (i - x * per_chunk);
                    if (u < u1) plan_recount(p, sh, u, hist, copies, lane);
                }
            }
            arrived = wait_for_all(p, sh.n_own, sh.arrived, &xq[1 + phase], n_chunks, tid);
            if (!arrived) break;
            // the part that holds the k-th largest
            plan_search(sh, p.n_cf, tid, [&](int j, const uint32_t*& h, uint32_t& nc, uint32_t& stride, const uint32_t*& extra, uint32_t& want) {
                h = hist + (size_t)j * copies * LCAP; nc = copies; stride = LCAP; extra = nullptr; want = sh.k[j] - sh.above[j];
            });
            if (tid < p.n_cf && sh.cut[tid]) {
                const uint32_t b = sh.fb[tid];
                if (b == NONE) { p.status->error = 1; sh.cut[tid] = 0; sh.mode[tid] = MODE_FAIL; }
                else {
                    sh.base[tid] += b << sh.s2[tid];
                    sh.above[tid] += sh.fa[tid];
                    sh.c[tid] = sh.fc[tid];
                    sh.bs[tid] = sh.s2[tid];
                    sh.mode[tid] = sh.bs[tid] == 0u ? MODE_RESOLVED : (sh.c[tid] <= (uint32_t)LCAP ? MODE_GATHER : MODE_FAIL);
                    sh.cut[tid] = sh.mode[tid] == MODE_FAIL ? 1u : 0u;
                    sh.s2[tid] = sh.bs[tid] > 11u ? sh.bs[tid] - 11u : 0u;
                }
            }
            __syncthreads();
            bool again = false;
            for (int j = 0; j < p.n_cf; ++j) again = again || sh.cut[j] != 0u;
            if (!again) break;
        }
        if (!arrived) {
            // whichever workgroup gives up records a plan that selects nothing inside the brackets: the later steps stay
            // inside their buffers, and the call's internal-error flag says that its results are not to be used
            counts = writes;
            writes = true;
            if (tid < p.n_cf) sh.mode[tid] = MODE_FAIL;
        }
    }
    if (!writes) return;
    if (tid < p.n_cf) {
        const int j = tid;
        CfState st;
        st.k = sh.k[j]; st.lo = sh.lo[j]; st.s = sh.s[j]; st.mode = sh.mode[j];
        st.base = 0; st.span = 0; st.above = 0; st.c = 0; st.tau = 0; st.need = 0; st.cnt_gt = 0; st.top = sh.top[j];
        st.pad[0] = st.pad[1] = st.pad[2] = st.pad[3] = 0;
        if (st.mode == MODE_FAIL) {
            p.status->error = 1;   // the exact routes cannot fail, except by giving up a wait
        } else {
            st.base = sh.base[j]; st.span = (1u << sh.bs[j]) - 1u; st.above = sh.above[j]; st.c = sh.c[j];
            if (st.mode == MODE_RESOLVED) { st.tau = st.base; st.cnt_gt = st.above; st.need = st.k - st.above; }
        }
        p.st[id0 + j] = st;
    }
    if (tid == 0) {
        // what the segment's tiles need of all its CFs together
        SegState sg;
        sg.fail = kind;
        sg.pz = kind == FAIL_FULL ? NONE : sh.pz;
        p.seg[t] = sg;
        if (kind >= FAIL_NARROW && counts) {
            p.status->any_fail = 1;
            atomicAdd(&p.status->n_fail, 1);
            if (kind == FAIL_NARROW) atomicAdd(&p.status->n_narrow, 1);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// R1: one wavefront per unit.  The unit's sums of the pass over the gradient (energy, entries above
// every CF's bracket and their energy) are added up over its sub-tiles; then the unit's entries inside
// the brackets are walked: per CF, those above the bin that holds the k-th largest are counted and
// their energy summed, those inside that bin are gathered (key, unit, value).
// ---------------------------------------------------------------------------------------------
// (the forms for three and four CFs are held to six wavefronts per SIMD: the ResNet101 shape's tiles are one round then)
// HEADS: the heads of the tile's lists are fetched before their lengths are known.  That pays where all tiles'
// wavefronts are resident at once and the kernel's time is one wavefront's chain of round trips to memory (the
// ResNet101 shape: 10.1 -> 7.9 us); with more tiles than that the chip is busy either way, and the extra loads and
// registers cost (the VGG16 shape: 10 -> 14 us), so the host picks the form by the number of tiles.
template <int NCF, bool HEADS, int U>  // compiled for calls with up to NCF CFs: the loops over the CFs are unrolled
__global__ __launch_bounds__(LWG) __attribute__((amdgpu_waves_per_eu((NCF == 3 || NCF == 4) ? 6 : 1, 8))) void refine_kernel(Params p)
{
    const int lane = threadIdx.x & 63;
    const uint32_t u = __builtin_amdgcn_readfirstlane(blockIdx.x * LWAVES + (threadIdx.x >> 6));
    if (u >= p.n_tiles * (SUB / U)) return;
    // loads that depend on nothing but the tile number come first, so that they are in flight together
    const double ssd = lane < U ? p.ssd[(size_t)u * U + lane] : 0.0;
    // ... among them the heads of the unit's lists, before their lengths are known: lane l takes entries
    // l % H + H r (r < SPEC_R) of sub-tile l / H, H = 64 / U.  A tile whose lists are no longer than that (most tiles of a call
    // with a CF of 100 or more) is done with one round trip to memory less.  Top-k keys only.
    constexpr int H = 64 / U, SPEC_R = HEADS ? (U == SUB ? 4 : U == MIDDLE ? 3 : 2) : 1;
    uint32_t spec[SPEC_R];
    if constexpr (HEADS) {
        const uint32_t* src = p.brk_key + (size_t)u * (U * TS) + (size_t)(lane / H) * TS + (lane % H);
#pragma unroll
        for (int r = 0; r < SPEC_R; ++r) spec[r] = src[H * r];
    }
    uint32_t on[NCF];
    double os[NCF];
#pragma unroll
    for (int j = 0; j < NCF; ++j) {
        const bool have = lane < U && j < p.n_cf;
        on[j] = have ? p.ovn[((size_t)u * U + lane) * p.n_cf + j] : 0u;
        os[j] = have ? p.ovs[((size_t)u * U + lane) * p.n_cf + j] : 0.0;
    }
    const int t = tile_seg(p, u / (SUB / U));
    // (the plan: fetched with the counts, not after them)
    uint32_t mode[NCF], base[NCF], span[NCF], top[NCF];
#pragma unroll
    for (int j = 0; j < NCF; ++j) {
        mode[j] = MODE_RESOLVED; base[j] = NONE; span[j] = 0; top[j] = 0;
        if (j < p.n_cf) {
            const CfState* st = &p.st[(size_t)t * p.n_cf + j];
            mode[j] = st->mode; base[j] = st->base; span[j] = st->span; top[j] = st->top;
        }
    }
    const UnitLists<U> tl = bracket_lists<U>(p, u);
    const uint32_t cnt = tl.total();
    uint32_t hn[NCF], tin = 0;
    double hs[NCF];
#pragma unroll
    for (int j = 0; j < NCF; ++j) { hn[j] = 0; hs[j] = 0.0; }
    if (cnt != 0) {
#pragma unroll
        for (int j = 0; j < NCF; ++j) {
            if (j < p.n_cf) {
                if (mode[j] == MODE_FAIL) { base[j] = NONE; top[j] = 0; }  // (an error: nothing is counted)
            }
        }
        // what one entry adds, per CF whose bracket it lies in (below top_j: what lies above was counted by the pass)
        const auto take = [&](uint32_t key, float val, bool live) {
            const double dv = p.random ? (double)val : (double)__uint_as_float(key);  // Top-k: the key is |acc|
#pragma unroll
            for (int j = 0; j < NCF; ++j) {
                if (j >= p.n_cf) continue;
                const bool mine = live && key < top[j] && key >= base[j];
                if (__ballot(mine) == 0ull) continue;  // (most rounds hold nothing for the CFs with few entries)
                const bool in = mine && key - base[j] <= span[j];
                // Random-k: the entry at the threshold is the last one selected and has no particular magnitude, so a
                // bin that is one key wide adds its energy here (Top-k adds need * tau^2 in the scan instead)
                if (mine && (!in || (p.random && mode[j] == MODE_RESOLVED))) { hs[j] += dv * dv; hn[j] += in ? 0u : 1u; }
                if (j == p.commit && in) ++tin;
                if (mode[j] == MODE_GATHER) {
                    // one counter update per wavefront: the lanes with a key in the bin take consecutive slots
                    const uint64_t m = __ballot(in);
                    if (m != 0ull) {
                        const size_t lst = seg_block(p, t, j) + (blockIdx.x & (seg_rep(p, t) - 1u));
                        const int leader = __ffsll((unsigned long long)m) - 1;
                        uint32_t at = 0;
                        if (lane == leader) at = atomicAdd(&p.list_cnt[lst * 32], (uint32_t)__popcll(m));
                        at = __shfl(at, leader, 64);
                        const uint32_t pos = at + lanes_below(m);
                        if (in && pos < LCAP) {
                            p.list_key[lst * LCAP + pos] = key;
                            p.list_tile[lst * LCAP + pos] = u;
                            if (p.random) p.list_val[lst * LCAP + pos] = val;
                        }
                    }
                }
            }
        };
        // 64 entries per load and lane-row, up to eight loads in flight per lane
        uint32_t i0 = 0;
        if constexpr (HEADS) {
            // the lists' heads cover the tile if every list is short enough
            bool heads = !p.random;
#pragma unroll
            for (int j = 0; j < U; ++j) heads = heads && tl.start[j + 1] - tl.start[j] <= (uint32_t)(H * SPEC_R);
            if (heads) {
                uint32_t mine_cnt = 0;
#pragma unroll
                for (int j = 0; j < U; ++j) if (lane / H == j) mine_cnt = tl.start[j + 1] - tl.start[j];
#pragma unroll 1
                for (int r = 0; r < SPEC_R; ++r) {
                    if (__ballot((uint32_t)(lane % H + H * r) < mine_cnt) == 0ull) break;
                    const uint32_t w = pop_front(spec);
                    take(w, 0.0f, (uint32_t)(lane % H + H * r) < mine_cnt);
                }
                i0 = cnt;
            }
        }
        if (i0 < cnt && cnt >= LONG_WALK && !p.random) {
            // long lists (a low CF, Top-k keys): sub-tile by sub-tile, so that no lane has to search for its entry's
            // slot.  A step's work is a fraction of a round trip to memory, and every wavefront of the launch is in
            // the same place, so the first two rounds of the next AHEAD sub-tiles are on their way while one is
            // worked on, whatever they hold; the words are carried as loaded and decoded where they are used
            // (decoded at once, the loads would be waited for at once).  The counts are the ones fetched with the
            // tile's first loads.
            constexpr int AHEAD = U < 4 ? U : 4;
            const auto fetch = [&](int j, uint32_t (&w)[2]) {
                const uint32_t* src = p.brk_key + (size_t)u * (U * TS) + (size_t)j * TS;
#pragma unroll
                for (int q = 0; q < 2; ++q) w[q] = src[q * 64 + lane];
            };
            uint32_t wq[AHEAD][2];
#pragma unroll
            for (int a = 0; a < AHEAD; ++a) fetch(a, wq[a]);
#pragma unroll 1
            for (int j = 0; j < U; ++j) {
                uint32_t w0[2], c = 0;
#pragma unroll
                for (int q = 0; q < 2; ++q) w0[q] = wq[0][q];
#pragma unroll
                for (int a = 0; a + 1 < AHEAD; ++a) { wq[a][0] = wq[a + 1][0]; wq[a][1] = wq[a + 1][1]; }
                if (j + AHEAD < U) fetch(j + AHEAD, wq[AHEAD - 1]);
#pragma unroll
                for (int x = 0; x < U; ++x) c = (x == j) ? tl.start[x + 1] - tl.start[x] : c;
                const uint32_t* src = p.brk_key + (size_t)u * (U * TS) + (size_t)j * TS;
#pragma unroll 1
                for (uint32_t b = 0; b < c; b += 64) {
                    const uint32_t w = w0[0];
                    w0[0] = w0[1];
                    if (b + 128 < c) w0[1] = src[(b + 128 + lane) & (TS - 1)];   // (the round after the next one)
                    take(w, 0.0f, b + lane < c);
                }
            }
            i0 = cnt;
        }
#pragma unroll 1
        for (; i0 < cnt; i0 += 64 * 8) {
            uint32_t kq[8];
            float vq[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                kq[q] = 0; vq[q] = 0.0f;
                if (i0 + q * 64 < cnt) {
                    const uint32_t i = i0 + q * 64 + lane;
                    const size_t at = (size_t)u * (U * TS) + tl.slot(i < cnt ? i : 0u);
                    kq[q] = p.brk_key[at];
                    if (p.random) vq[q] = p.brk_val[at];
                }
            }
#pragma unroll 1
            for (uint32_t i = i0; i < i0 + 64 * 8 && i < cnt; i += 64) {
                const uint32_t key = pop_front(kq);
                const float val = pop_front(vq);
                take(key, val, i + lane < cnt);
            }
        }
    }
    // zeros that the pass has counted and not listed are inside the located bin if that is theirs alone
#pragma unroll
    for (int j = 0; j < NCF; ++j)
        if (j < p.n_cf && j == p.commit && mode[j] == MODE_RESOLVED && base[j] == 0u && lane == 0) tin += tl.zeros;
    // the tile's sums: what the pass over the gradient counted above the brackets, plus the above
    {
        const double x = wave_sum(ssd);
        if (lane == 0) p.ssd_t[u] = x;
    }
    tin = wave_sum(tin);
#pragma unroll
    for (int j = 0; j < NCF; ++j) {
        if (j < p.n_cf) {
            const uint32_t n = wave_sum(hn[j] + on[j]);
            // (the counted energy first, in sub-tile order, then the listed entries': a fixed order)
            const double e = wave_sum(os[j]) + wave_sum(hs[j]);
            if (lane == 0) {
                p.sss[(size_t)u * p.n_cf + j] = e;
                if (j == p.commit) {
                    p.tg0[u] = n; p.tin[u] = tin;
                    if (p.csum) atomicAdd((unsigned long long*)&p.csum[(size_t)(u / CTILES) * 8], ((unsigned long long)n << 32) | tin);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// SCAN: grid (n_seg, slices + n_cf), SCAN_T threads.  Every block first resolves one CF of its segment to
//       the exact key tau of the k-th largest (from the gathered keys by a bitwise search), and how many keys equal to
//       tau are selected.
//       Block (t, y < slices), committed CF: the counts of the y-th slice of SCAN_SLICE tiles of
//       segment t (entries above the located bin, plus the gathered entries above tau, by tile) and their
//       exclusive scan -> every tile's output offset and tie quota.  The totals of the earlier slices are
//       re-added by every block (a few batched loads), so no block waits on another.
//       Block (t, slices + j): statistics of (segment t, CF j), summed over the tiles in a fixed order.
// ---------------------------------------------------------------------------------------------
constexpr int SCAN_T = 1024;                 // threads
constexpr int SCAN_W = SCAN_T / 64;
constexpr int SCAN_PER = 4;                  // tiles per thread
constexpr int SCAN_SLICE = SCAN_T * SCAN_PER;
constexpr int LPER = LCAP / SCAN_T;          // gathered entries per thread
constexpr int RW = LPER;
constexpr int SCAN_SPEC = SCAN_T / REP;      // threads that fetch the head of one gather list before its length is known
static_assert(LCAP % SCAN_T == 0 && SCAN_T % REP == 0 && SCAN_SPEC * LPER <= LCAP && 2 * SCAN_T == NBIN,
              "the gathered entries are dealt evenly; a thread owns two bins of the search's histogram");

__global__ __launch_bounds__(SCAN_T) void scan_kernel(Params p, uint32_t slices)
{
    __shared__ uint32_t sg[SCAN_SLICE], se[SCAN_SLICE];
    __shared__ uint32_t wt[4][SCAN_W];
    __shared__ uint32_t wsum[2][SCAN_W];
    __shared__ double dred[3][SCAN_W];
    __shared__ uint64_t ured[SCAN_W];
    __shared__ uint32_t res3[3];
    const int tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    const int t = blockIdx.x;
    const bool scan_role = blockIdx.y < slices;
    const int j = scan_role ? p.commit : (int)(blockIdx.y - slices);
    const uint32_t id = (uint32_t)t * p.n_cf + j;
    const uint32_t u0 = seg_tile0(p, t), u1 = seg_tile1(p, t);
    const uint32_t slice0 = scan_role ? u0 + blockIdx.y * SCAN_SLICE : 0u;
    if ((scan_role && slice0 >= u1) || seg_small(p, t)) return;
    CfState* st = &p.st[id];

    // ---- loads that do not depend on the threshold come first, so that they overlap with its resolution
    // the fill counts of the gather lists and the plan
    const uint32_t copies = seg_rep(p, t);
    const size_t block0 = seg_block(p, t, j);
    uint32_t fill[REP];
#pragma unroll
    for (int r = 0; r < REP; ++r) fill[r] = (uint32_t)r < copies ? p.list_cnt[(block0 + r) * 32] : 0u;
    const uint32_t mode = st->mode, k = st->k, above = st->above, base = st->base, span = st->span, c = st->c;
    uint32_t tau = st->tau, need = st->need, cnt_gt = st->cnt_gt;   // valid if the located bin was one key wide
    // ... and the head of every gather list, SCAN_SPEC * LPER entries of it, before the fill counts are known: a list is
    // rarely longer than that (the located bin's entries spread over the copies), and a load that waits for the
    // counts would cost this kernel another round trip to memory
    const uint32_t spec_r = (uint32_t)tid / SCAN_SPEC;
    uint32_t sk[LPER], stl[LPER];
    float sv[LPER];
#pragma unroll
    for (int q = 0; q < LPER; ++q) {
        const size_t at = (block0 + (spec_r < copies ? spec_r : 0u)) * LCAP + (uint32_t)(tid % SCAN_SPEC) + (uint32_t)q * SCAN_SPEC;
        sk[q] = p.list_key[at];
        stl[q] = p.list_tile[at];
        sv[q] = p.random ? p.list_val[at] : 0.0f;
    }
    // scan: this slice, coalesced (entries above the located bin, entries inside it), and the totals of the
    // earlier slices of this segment; statistics: the tiles' sums, sixteen tiles per thread and round, fixed order
    uint32_t og[SCAN_PER], oi[SCAN_PER], pg = 0, pi = 0;
    double sd = 0.0, sj = 0.0;
    if (scan_role) {
#pragma unroll
        for (int q = 0; q < SCAN_PER; ++q) {
            const uint32_t u = slice0 + q * SCAN_T + tid;
            og[q] = (u < u1) ? p.tg0[u] : 0u;
            oi[q] = (u < u1) ? p.tin[u] : 0u;
        }
        for (uint32_t v0 = u0 + tid; v0 < slice0; v0 += 32 * SCAN_T) {
            uint32_t xg[32], xe[32];
#pragma unroll
            for (int q = 0; q < 32; ++q) {
                const uint32_t v = v0 + q * SCAN_T;
                xg[q] = (v < slice0) ? p.tg0[v] : 0u;
                xe[q] = (v < slice0) ? p.tin[v] : 0u;
            }
#pragma unroll
            for (int q = 0; q < 32; ++q) { pg += xg[q]; pi += xe[q]; }
        }
    } else {
        for (uint32_t v0 = u0 + tid; v0 < u1; v0 += 16 * SCAN_T) {
            double xd[16], xj[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const uint32_t u = v0 + q * SCAN_T;
                xd[q] = (u < u1) ? p.ssd_t[u] : 0.0;
                xj[q] = (u < u1) ? p.sss[(size_t)u * p.n_cf + j] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) { sd += xd[q]; sj += xj[q]; }
        }
    }

    // ---- resolve (segment t, CF j)
    // This thread's gathered entries: key - base, tile, value, and which of the slots hold one (LPER per thread).
    uint32_t d[RW], rt[RW], live = 0;
    float rv[RW];
#pragma unroll
    for (int q = 0; q < RW; ++q) { d[q] = 0; rt[q] = 0; rv[q] = 0.0f; }
    if (mode == MODE_FAIL) {
        if (tid == 0) p.status->error = 1;
        tau = 0; need = 0; cnt_gt = 0;
    } else if (mode == MODE_GATHER) {
        // the want-th largest of the listed keys d = key - base.
        // The keys sit in REP lists; list r holds positions [off_r, off_r + n_r) of the concatenation.
        const uint32_t want = k - above;
        uint32_t off[REP + 1];
        off[0] = 0;
#pragma unroll
        for (int r = 0; r < REP; ++r) off[r + 1] = off[r] + fill[r];
        if (off[REP] != c || c > LCAP || want == 0 || want > c) {
            if (tid == 0) p.status->error = 1;
            tau = base; need = 0; cnt_gt = above;
        } else {
            bool spec_ok = true;
#pragma unroll
            for (int r = 0; r < REP; ++r) spec_ok = spec_ok && fill[r] <= (uint32_t)(SCAN_SPEC * LPER);
            if (spec_ok) {
                // the entries are the ones fetched ahead: list spec_r, slots tid % SCAN_SPEC + q SCAN_SPEC
                uint32_t my_fill = 0;
#pragma unroll
                for (int r = 0; r < REP; ++r) if ((uint32_t)r == spec_r) my_fill = fill[r];   // (0 beyond the segment's copies)
#pragma unroll
                for (int q = 0; q < LPER; ++q) {
                    const uint32_t slot = (uint32_t)(tid % SCAN_SPEC) + (uint32_t)q * SCAN_SPEC;
                    d[q] = sk[q]; rt[q] = stl[q]; rv[q] = sv[q];
                    if (slot < my_fill) live |= 1u << q;
                }
            } else {
                // a long list: the entries are dealt over the block by their position in the concatenation; all loads
                // first, without branches around them (a position past the last key reads key 0 of the lists instead;
                // c >= 1 here), so that they are in flight together
#pragma unroll
                for (int q = 0; q < LPER; ++q) {
                    const uint32_t pos = (uint32_t)(q * SCAN_T + tid);
                    const uint32_t i = pos < c ? pos : 0u;
                    int r = 0;
#pragma unroll
                    for (int x = 1; x < REP; ++x) r += (i >= off[x]);
                    uint32_t o = 0;
#pragma unroll
                    for (int x = 0; x < REP; ++x) if (x == r) o = off[x];
                    const size_t at = (block0 + r) * LCAP + (i - o);
                    d[q] = p.list_key[at];
                    rt[q] = p.list_tile[at];
                    rv[q] = p.random ? p.list_val[at] : 0.0f;
                    if (pos < c) live |= 1u << q;
                }
            }
#pragma unroll
            for (int q = 0; q < LPER; ++q) d[q] = ((live >> q) & 1u) ? d[q] - base : 0u;
            // The want-th largest d: a histogram of 11 bits of d at a time, from the top bits down (one round unless
            // the located bin is more than 2048 keys wide), among the entries that agree with the bits found so far.
            // Thread tid owns bins 2047 - 2 tid and 2046 - 2 tid, so that a scan over the threads runs from the top bin.
            int nbits = 0;
            while (nbits < 32 && (span >> nbits) != 0u) ++nbits;
            uint32_t prefix = 0, pmask = 0, gsum = 0, left = want;
            int shift = nbits > 11 ? nbits - 11 : 0;
            for (;;) {
                sg[2 * tid] = 0; sg[2 * tid + 1] = 0;
                __syncthreads();
#pragma unroll
                for (int q = 0; q < LPER; ++q)
                    if (((live >> q) & 1u) && (d[q] & pmask) == prefix) atomicAdd(&sg[(d[q] >> shift) & (NBIN - 1)], 1u);
                __syncthreads();
                const uint32_t bA = (uint32_t)(NBIN - 1 - 2 * tid), bB = bA - 1u;
                const uint32_t hA = sg[bA], hB = sg[bB], mine = hA + hB;
                const uint32_t incl = wave_scan(mine);
                if (lane == 63) wsum[0][wib] = incl;
                __syncthreads();
                uint32_t higher = incl - mine;   // entries in the bins above this thread's two
#pragma unroll
                for (int w = 0; w < SCAN_W; ++w) if (w < wib) higher += wsum[0][w];
                if (higher < left && higher + hA >= left) { res3[0] = bA; res3[1] = higher; }
                else if (higher + hA < left && higher + mine >= left) { res3[0] = bB; res3[1] = higher + hA; }
                __syncthreads();
                prefix |= res3[0] << shift;
                pmask |= (uint32_t)(NBIN - 1) << shift;
                gsum += res3[1];
                left -= res3[1];
                if (shift == 0) break;
                shift = shift > 11 ? shift - 11 : 0;
                __syncthreads();   // (res3 and the histogram are rewritten in the next round)
            }
            tau = base + prefix; cnt_gt = above + gsum; need = k - cnt_gt;
            __syncthreads();
        }
    }
    const uint32_t dtau = tau - base;  // the threshold inside the located bin

    if (scan_role) {
        // (the plan itself stays as it is: the segment's other blocks are reading it)
        if (blockIdx.y == 0 && tid == 0) { st->tau = tau; st->need = need; st->cnt_gt = cnt_gt; }
        // entries equal to tau: those inside a located bin that is one key wide
        uint32_t pe = (mode == MODE_RESOLVED) ? pi : 0u;
#pragma unroll
        for (int q = 0; q < SCAN_PER; ++q) {
            sg[q * SCAN_T + tid] = og[q];
            se[q * SCAN_T + tid] = (mode == MODE_RESOLVED) ? oi[q] : 0u;
        }
        __syncthreads();
        if (mode == MODE_GATHER) {
            // the gathered entries above and at the threshold, by tile
#pragma unroll
            for (int q = 0; q < RW; ++q) {
                if (!((live >> q) & 1u) || d[q] < dtau) continue;
                const bool gt = d[q] > dtau;
                if (rt[q] < slice0) { if (gt) ++pg; else ++pe; }
                else if (rt[q] - slice0 < (uint32_t)SCAN_SLICE) atomicAdd(gt ? &sg[rt[q] - slice0] : &se[rt[q] - slice0], 1u);
            }
        }
        pg = wave_sum(pg);
        pe = wave_sum(pe);
        if (lane == 0) { wt[2][wib] = pg; wt[3][wib] = pe; }
        __syncthreads();
        // this thread's SCAN_PER consecutive tiles
        uint32_t g[SCAN_PER], e[SCAN_PER], sum_g = 0, sum_e = 0;
#pragma unroll
        for (int i = 0; i < SCAN_PER; ++i) {
            g[i] = sg[tid * SCAN_PER + i]; e[i] = se[tid * SCAN_PER + i];
            sum_g += g[i]; sum_e += e[i];
        }
        const uint32_t ig = wave_scan(sum_g), ie = wave_scan(sum_e);
        if (lane == 63) { wt[0][wib] = ig; wt[1][wib] = ie; }
        __syncthreads();
        uint32_t run_g = ig - sum_g, run_e = ie - sum_e;   // counts before this thread's tiles
#pragma unroll
        for (int w = 0; w < SCAN_W; ++w) {
            if (w < wib) { run_g += wt[0][w]; run_e += wt[1][w]; }
            run_g += wt[2][w];
            run_e += wt[3][w];
        }
        uint32_t off[SCAN_PER], tk[SCAN_PER];
#pragma unroll
        for (int i = 0; i < SCAN_PER; ++i) {
            const uint32_t ties_before = run_e < need ? run_e : need;  // ties selected in earlier tiles
            const uint32_t left = need - ties_before;
            off[i] = run_g + ties_before;                               // output offset of the tile
            tk[i] = left < e[i] ? left : e[i];                          // its tie quota
            run_g += g[i];
            run_e += e[i];
        }
        // the number of pairs a tile emits is written by the thread that holds its counts
#pragma unroll
        for (int i = 0; i < SCAN_PER; ++i) {
            const uint32_t u = slice0 + tid * SCAN_PER + i;
            if (u < u1) p.tsel[u] = g[i] + tk[i];
        }
        // threshold sparsifier: how many entries are kept is only known here (the last thread of the last slice has
        // counted them all); the emit step emits them if they fit the caller's buffers
        if (p.bounds_from == BOUNDS_FIXED && tid == SCAN_T - 1 && slice0 + SCAN_SLICE >= u1) {
            p.status->count = (int)run_g;
            if (p.out_count) *p.out_count = (int64_t)run_g;
        }
#pragma unroll
        for (int i = 0; i < SCAN_PER; ++i) {
            sg[tid * SCAN_PER + i] = off[i];
            se[tid * SCAN_PER + i] = tk[i];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < SCAN_PER; ++q) {
            const uint32_t u = slice0 + q * SCAN_T + tid;
            if (u < u1) { p.toff[u] = sg[q * SCAN_T + tid]; p.ttake[u] = se[q * SCAN_T + tid]; }
        }
        return;
    }

    // ---- statistics of (segment t, CF j)
    // the entries of the located bin above the threshold (Random-k: and the one at it).  Their order in the gather
    // lists varies from run to run, so their energies are added as integers: every square, exact in binary64, is
    // scaled by a power of two that puts the largest of them below 2^50 and truncated, the sum of up to LCAP of them
    // fits 64 bits and does not depend on the order, and it is off by less than 2^-38 of itself.
    double ebin = 0.0;
    if (mode == MODE_GATHER) {
        const auto square = [&](int q) {
            const bool in = ((live >> q) & 1u) && (d[q] > dtau || (p.random && d[q] == dtau));
            const double dv = p.random ? (double)rv[q] : (double)__uint_as_float(base + d[q]);
            return in ? dv * dv : 0.0;
        };
        const uint32_t kmax = base + span;   // the located bin's largest key
        if (!p.random && kmax < 0x7F800000u) {
            // Top-k keys are magnitudes, and the bin's own bounds say how large a square can get: no look at the
            // entries for the scale, and nothing can be infinite or NaN
            if (kmax != 0u) {
                const double m = (double)__uint_as_float(kmax);
                const int ex = ilogb(m * m);                  // every square is below 2^(ex + 1)
                const double sc = scalbn(1.0, 49 - ex);       // (a power of two: the product is exact)
                uint64_t acc = 0;
#pragma unroll
                for (int q = 0; q < RW; ++q) acc += (uint64_t)(square(q) * sc);   // < 2^50 each
                acc = wave_sum(acc);
                if (lane == 0) ured[wib] = acc;
                __syncthreads();
                uint64_t all = 0;
#pragma unroll
                for (int w = 0; w < SCAN_W; ++w) all += ured[w];
                ebin = scalbn((double)all, ex - 49);
            }
        } else {
        double mx = 0.0, plain = 0.0;
        bool finite = true;
#pragma unroll
        for (int q = 0; q < RW; ++q) {
            const double x = square(q);
            mx = fmax(mx, x);   // (a NaN square is skipped here and shows in the plain sum)
            plain += x;
            finite = finite && (x <= 1.0e300);
        }
        mx = wave_max(mx);
        if (lane == 0) dred[2][wib] = mx;
        const bool all_finite = __syncthreads_and(finite ? 1 : 0) != 0;
        mx = 0.0;
#pragma unroll
        for (int w = 0; w < SCAN_W; ++w) mx = fmax(mx, dred[2][w]);
        __syncthreads();
        if (!all_finite) {
            // an infinite or NaN square: the sum is infinite or NaN in any order
            plain = wave_sum(plain);
            if (lane == 0) dred[2][wib] = plain;
            __syncthreads();
            for (int w = 0; w < SCAN_W; ++w) ebin += dred[2][w];
        } else if (mx > 0.0) {
            const int ex = ilogb(mx);                      // 2^ex <= mx < 2^(ex + 1)
            uint64_t acc = 0;
#pragma unroll
            for (int q = 0; q < RW; ++q) acc += (uint64_t)scalbn(square(q), 49 - ex);   // < 2^50 each
            acc = wave_sum(acc);
            if (lane == 0) ured[wib] = acc;
            __syncthreads();
            uint64_t all = 0;
#pragma unroll
            for (int w = 0; w < SCAN_W; ++w) all += ured[w];
            ebin = scalbn((double)all, ex - 49);
        }
        }
    }
    // every wavefront's sum, then the SCAN_W of them in order: the same order in every run
    {
        const double wd = wave_sum(sd), wj = wave_sum(sj);
        if (lane == 0) { dred[0][wib] = wd; dred[1][wib] = wj; }
    }
    __syncthreads();
    if (tid == 0) {
        // fourth statistic: the threshold as a magnitude (Top-k) or as a priority (Random-k)
        const double tauv = p.random ? (double)tau : (double)__uint_as_float(tau);
        double ss_dense = 0.0, ss_above = 0.0;
        for (int w = 0; w < SCAN_W; ++w) { ss_dense += dred[0][w]; ss_above += dred[1][w]; }
        // Top-k: the ties all have magnitude tau; Random-k: the entry at the threshold has been summed
        const double ss_sel = ss_above + ebin + (p.random ? 0.0 : (double)need * tauv * tauv);
        double* o = p.out_stats + (size_t)id * GRAVAC_STATS_PER_CF;
        o[0] = ss_sel;
        o[1] = ss_dense;
        o[2] = (ss_dense == 0.0) ? 1.0 : ss_sel / ss_dense;
        o[3] = p.bounds_from == BOUNDS_FIXED ? (double)__uint_as_float(p.fixed_key) : tauv;
        if (j != p.commit) { st->tau = tau; st->need = need; st->cnt_gt = cnt_gt; }
    }
}

// ---------------------------------------------------------------------------------------------
// EMIT: the tiles' shares of the committed selection in ascending index order, a wavefront per tile, and zeroes in its
//       residual slots.  A sub-tile with a candidate list is emitted from the list; a sub-tile without one (mostly
//       candidates) is read again, 1024 elements, and its residual rewritten.  Two kernels:
//
// emit_kernel works from what the scan step has left.
//
// resolve_emit_kernel does the scan step's work itself: every workgroup resolves the committed CF of its segment to the
// exact key tau of the k-th largest from the gathered entries, and adds up what lies before its eight units (totals of 64
// units each, which the refine step has added up, and up to 126 single tiles at the ends).  The first n_seg n_cf workgroups
// of its launch are the statistics of one (segment, CF) each.  The scan step is 6 to 8 us of round trips and barriers in
// one or a few workgroups; repeated by all of them, part of it overlaps with the tiles' own first loads, and a launch is
// spared: 1 MiB buckets 38.3 -> 33.8 us, 25 MB 74.7 -> 72.4, ResNet101 CF 100 129.9 -> 126.3, three CFs 197 -> 192, LSTM
// 156 -> 151 (with the rolled loops of pop_front, which took 1 to 3 us of that).  It holds while all tiles' wavefronts are
// resident at once (EMIT_RESIDENT: six per SIMD); the VGG16 shape's 2112 workgroups take two to three rounds of it, 386
// instead of 381 us at CF 1000 and 439 instead of 417 at CF 10, and stay with the scan step.  (Normal gradients of 50 to 100
// million elements: within 1.5 % either way, 137.8 against 138.8 us just below the limit and 139.4 against 140.5 just above.)
// ---------------------------------------------------------------------------------------------
constexpr int EWG = 512;                    // threads
constexpr int EW = EWG / 64;
constexpr uint32_t WIDE_CHUNKS = (uint32_t)(DIRECT_MAX / (EW * FINE * TS));   // chunks of EW units of a direct call at most
static_assert(DIRECT_MAX % (EW * FINE * TS) == 0 && DIRECT_MAX % TW == 0, "its units are whole chunks");
constexpr uint32_t EMIT_RESIDENT = 6144;    // tiles (six wavefronts on each of 1024 SIMDs)
constexpr int SPEC = EWG / REP;             // threads that fetch the head of one gather list before its length is known,
constexpr int SPEC_Q = 2;                   // ... SPEC_Q entries each
static_assert(EWG % REP == 0 && SPEC * SPEC_Q <= LCAP && 4 * EWG == NBIN, "a thread owns four bins of the search's histogram");

struct EmitShared {
    uint32_t hist[NBIN];
    uint32_t wsum[EW];
    uint32_t pick[2];
    uint32_t fg[EW], fe[EW];                // gathered entries above / at the threshold, per tile of the workgroup
    uint32_t tg[EW], te[EW];                // the tiles' counts, as refine_kernel leaves them
    uint32_t ws[3][EW];
    double dred[3][EW];
    uint64_t ured[EW];
};

// A direct call's bins that are cut again, as they are then (wide_resolve).
struct WideShared {
    uint32_t mode[MAXCF], base[MAXCF], span[MAXCF], above[MAXCF], c[MAXCF];
    uint32_t in;                            // entries in the bin that pick_bin has found
    uint32_t got, n_own, arrived;
    uint32_t own[WIDE_CHUNKS];              // the chunks of units this workgroup has claimed
};

// The located bin of one (segment, CF) and the entries gathered from it.
struct Gathered {
    uint32_t mode, k, above, base, span, c;
    uint32_t tau, need, cnt_gt;             // the result
    uint32_t fill[REP];
    size_t block0;                          // first copy block
    uint32_t sk[SPEC_Q], stl[SPEC_Q];       // heads of the lists
    float sv[SPEC_Q];
    uint32_t my_fill;                       // entries in the list whose head this thread has fetched
    bool spec;                              // the heads are all there is
};

// The loads that start a resolution; the heads of the gather lists come before their fill counts are known: a list is
// rarely longer than that (the located bin's entries spread over the copies), and a load that waits for the counts
// would cost another round trip to memory.
__device__ __forceinline__ void gathered_load(const Params& p, int t, int j, int tid, Gathered& g)
{
    const uint32_t copies = seg_rep(p, t);
    g.block0 = seg_block(p, t, j);
    const CfState* st = &p.st[(size_t)t * p.n_cf + j];
#pragma unroll
    for (int r = 0; r < REP; ++r) g.fill[r] = (uint32_t)r < copies ? p.list_cnt[(g.block0 + r) * 32] : 0u;
    const uint32_t r = (uint32_t)tid / SPEC;
#pragma unroll
    for (int q = 0; q < SPEC_Q; ++q) {
        const size_t at = (g.block0 + (r < copies ? r : 0u)) * LCAP + (uint32_t)(tid % SPEC) + (uint32_t)q * SPEC;
        g.sk[q] = p.list_key[at];
        g.stl[q] = p.list_tile[at];
        g.sv[q] = p.random ? p.list_val[at] : 0.0f;
    }
    g.mode = st->mode; g.k = st->k; g.above = st->above; g.base = st->base; g.span = st->span; g.c = st->c;
    g.tau = st->tau; g.need = st->need; g.cnt_gt = st->cnt_gt;   // valid if the located bin was one key wide
    bool spec = true;
    uint32_t mine = 0;
#pragma unroll
    for (int x = 0; x < REP; ++x) {
        spec = spec && g.fill[x] <= (uint32_t)(SPEC * SPEC_Q);
        if ((uint32_t)x == r) mine = g.fill[x];   // (0 beyond the segment's copies)
    }
    g.spec = spec;
    g.my_fill = mine;
}

// f(key - base, tile, value) for every gathered entry of this thread.
template <typename F>
__device__ __forceinline__ void gathered_each(const Params& p, int tid, const Gathered& g, F f)
{
    if (g.spec) {
#pragma unroll
        for (int q = 0; q < SPEC_Q; ++q)
            if ((uint32_t)(tid % SPEC) + (uint32_t)q * SPEC < g.my_fill) f(g.sk[q] - g.base, g.stl[q], g.sv[q]);
        return;
    }
    // a long list: the entries are dealt over the workgroup by their position in the concatenation
    for (uint32_t pos = tid; pos < g.c; pos += EWG) {
        uint32_t r = 0, before = 0, sum = 0;
#pragma unroll
        for (int x = 0; x < REP; ++x) {
            if (pos >= sum) { r = x; before = sum; }
            sum += g.fill[x];
        }
        const size_t at = (g.block0 + r) * LCAP + (pos - before);
        f(p.list_key[at] - g.base, p.list_tile[at], p.random ? p.list_val[at] : 0.0f);
    }
}

// The bin of the left-th largest entry of a histogram of which thread tid holds bins 2044 - 4 tid .. 2047 - 4 tid: sh.pick is
// the bin and what lies above it, *in what is in it.
__device__ __forceinline__ void pick_bin(EmitShared& sh, const uint4& hv, uint32_t left, int tid, uint32_t* in = nullptr)
{
    const int lane = tid & 63, wib = tid >> 6;
    const uint32_t hh[4] = {hv.w, hv.z, hv.y, hv.x}, mine = hv.x + hv.y + hv.z + hv.w;
    const uint32_t incl = wave_scan(mine);
    if (lane == 63) sh.wsum[wib] = incl;
    __syncthreads();
    uint32_t higher = incl - mine;   // entries in the bins above this thread's four
#pragma unroll
    for (int w = 0; w < EW; ++w) if (w < wib) higher += sh.wsum[w];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (higher < left && higher + hh[e] >= left) {
            sh.pick[0] = (uint32_t)(NBIN - 1 - 4 * tid - e);
            sh.pick[1] = higher;
            if (in) *in = hh[e];
        }
        higher += hh[e];
    }
    __syncthreads();
}

// g.tau / need / cnt_gt: the key of the k-th largest, how many equal to it are selected, how many lie above.
__device__ __forceinline__ void gathered_resolve(const Params& p, int tid, Gathered& g, EmitShared& sh)
{
    if (g.mode == MODE_RESOLVED) return;
    uint32_t filled = 0;
#pragma unroll
    for (int r = 0; r < REP; ++r) filled += g.fill[r];
    const uint32_t want = g.k - g.above;
    if (g.mode != MODE_GATHER || filled != g.c || g.c > (uint32_t)LCAP || want == 0 || want > g.c) {
        if (tid == 0) p.status->error = 1;
        g.mode = MODE_FAIL;
        g.tau = g.base; g.need = 0; g.cnt_gt = g.above;
        return;
    }
    // The want-th largest d = key - base: a histogram of 11 bits of d at a time, from the top bits down (one round unless
    // the located bin is more than 2048 keys wide), among the entries that agree with the bits found so far.
    // Thread tid owns bins 2047 - 4 tid .. 2044 - 4 tid, so that a scan over the threads runs from the top bin.
    int nbits = 0;
    while (nbits < 32 && (g.span >> nbits) != 0u) ++nbits;
    uint32_t prefix = 0, pmask = 0, gsum = 0, left = want;
    int shift = nbits > 11 ? nbits - 11 : 0;
    for (;;) {
        *(uint4*)&sh.hist[4 * tid] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        gathered_each(p, tid, g, [&](uint32_t d, uint32_t, float) {
            if ((d & pmask) == prefix) atomicAdd(&sh.hist[(d >> shift) & (NBIN - 1)], 1u);
        });
        __syncthreads();
        pick_bin(sh, *(const uint4*)&sh.hist[NBIN - 4 - 4 * tid], left, tid);
        prefix |= sh.pick[0] << shift;
        pmask |= (uint32_t)(NBIN - 1) << shift;
        gsum += sh.pick[1];
        left -= sh.pick[1];
        if (shift == 0) break;
        shift = shift > 11 ? shift - 11 : 0;
        __syncthreads();   // (pick is rewritten in the next round)
    }
    g.tau = g.base + prefix; g.cnt_gt = g.above + gsum; g.need = g.k - g.cnt_gt;
}

// A direct call whose pass has found bins too full to gather or too wide (a mass of equal values, magnitudes close together, a
// second part of the tensor far from the finely binned octaves).  All workgroups of the emit step, the statistics' among them,
// cut them together before they do anything else, as the plan step does on its exact routes and with the same kind of queue: the
// units are claimed in chunks, a workgroup waits for chunks that running workgroups have claimed and for nothing else.  Per such
// CF a histogram of 11 bits of the bin's keys from the bracket lists, until what holds the k-th largest is one key or little
// enough to gather; then a walk that counts and sums up, per unit, what lies above that, and gathers what lies inside.
// (524,288 elements, magnitudes within 10 % of each other, CF 100, and within 1 %; 255 values, CF 10; one value, CF 100: 39, 44, 41
// and 73 us.  Resolved by every workgroup for itself from all lists: 253, 312, 184 and 924; by the plan and refine steps, two launches
// more for every call: 37, 51, 78 and 820.)
template <int U>
__device__ __forceinline__ void wide_resolve(const Params& p, int tid, EmitShared& sh, WideShared& ws)
{
    const int lane = tid & 63, wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t units = p.n_tiles * (SUB / U), n_chunks = (units + EW - 1u) / EW;
    uint32_t waits = 0;
    bool arrived = true;
    if (tid == 0) ws.n_own = 0;
    if (tid < p.n_cf) {
        const CfState* st = &p.st[tid];
        ws.mode[tid] = st->mode; ws.base[tid] = st->base; ws.span[tid] = st->span;
        ws.above[tid] = st->above; ws.c[tid] = st->c;
    }
    // f(key, live) for the listed entries of unit u, by all lanes of a wavefront
    const auto walk = [&](uint32_t u, auto f) {
        const UnitLists<U> tl = bracket_lists<U>(p, u);
        constexpr uint32_t K = 8;   // loads in flight
#pragma unroll 1
        for (int i = 0; i < U; ++i) {
            uint32_t n = 0;
#pragma unroll
            for (int x = 0; x < U; ++x) n = x == i ? tl.start[x + 1] - tl.start[x] : n;
            const uint32_t* src = p.brk_key + ((size_t)u * U + i) * TS + lane;
#pragma unroll 1
            for (uint32_t b = 0; b < n; b += 64 * K) {   // (a list's slots are a multiple of that; those past its end are not used)
                static_assert(TS % (64 * K) == 0, "inside the sub-tile's slots");
                uint32_t k[K];
#pragma unroll
                for (uint32_t q = 0; q < K; ++q) k[q] = src[b + 64 * q];
#pragma unroll 1
                for (uint32_t x = b; x < b + 64 * K && x < n; x += 64) {
                    const uint32_t key = pop_front(k);
                    f(key, x + lane < n);
                }
            }
        }
    };
    bool first = true;
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < p.n_cf && arrived; ++j) {
        if (ws.mode[j] != MODE_WIDE) continue;
        const uint32_t k = p.flat_k[j];
        uint32_t base = ws.base[j], span = ws.span[j], above = ws.above[j], c = ws.c[j];
#pragma unroll 1
        for (uint32_t round = 0; round < WIDE_ROUNDS; ++round) {
            // (keys of denormal numbers lie octaves apart: they are cut down to one)
            if (span == 0u || (c <= (uint32_t)LCAP && span < (1u << SCSHIFT) && base >= 0x00800000u)) break;
            const uint32_t nbits = 32u - (uint32_t)__clz((int)span), shift = nbits > 11u ? nbits - 11u : 0u;
            *(uint4*)&sh.hist[4 * tid] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
            const auto count = [&](uint32_t u) {
                walk(u, [&](uint32_t key, bool live) {
                    const bool in = live && key >= base && key - base <= span;
                    const uint32_t bin = (key - base) >> shift;
                    // a mass of equal keys: the lanes that share the first one's bin add once
                    const uint64_t m = __ballot(in);
                    if (m == 0ull) return;
                    const int leader = __ffsll((unsigned long long)m) - 1;
                    const uint64_t same = __ballot(in && bin == (uint32_t)__shfl((int)bin, leader, 64));
                    if (lane == leader) atomicAdd(&sh.hist[bin], (uint32_t)__popcll(same));
                    else if (in && !((same >> lane) & 1ull)) atomicAdd(&sh.hist[bin], 1u);
                });
            };
            if (first) {
                // The chunks are claimed as they are worked on.  (The last thing of a round is a barrier for everybody.  With a
                // statement of thread 0 there the compiler joins it with the one that the next round begins with, for which
                // the other lanes of its wavefront then do not wait: they go round without it, for ever.)
                first = false;
                for (;;) {
                    if (tid == 0) {
                        ws.got = ws.n_own < WIDE_CHUNKS ? atomicAdd(&p.xq[0], 1u) : NONE;   // (there are no more than that)
                        if (ws.got < n_chunks) ws.own[ws.n_own++] = ws.got;
                    }
                    __syncthreads();
                    const uint32_t at = ws.got;
                    if (at >= n_chunks) break;
                    const uint32_t u = __builtin_amdgcn_readfirstlane(at * EW + wib);
                    if (u < units) count(u);
                    __syncthreads();
                }
            } else {
                for (uint32_t x = 0; x < ws.n_own; ++x) {
                    const uint32_t u = __builtin_amdgcn_readfirstlane(ws.own[x] * EW + wib);
                    if (u < units) count(u);
                }
            }
            __syncthreads();
            uint32_t* all = wide_hist(p, j, round);
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const uint32_t x = sh.hist[4 * tid + e];
                if (x != 0u) atomicAdd(&all[4 * tid + e], x);
            }
            arrived = wait_for_all(p, ws.n_own, ws.arrived, &p.xq[1], ++waits * n_chunks, tid);
            if (!arrived) break;
            if (tid == 0) sh.pick[0] = NONE;
            __syncthreads();
            pick_bin(sh, *(const uint4*)&all[NBIN - 4 - 4 * tid], k - above, tid, &ws.in);
            const uint32_t b = sh.pick[0];
            if (b == NONE) { arrived = false; break; }   // cannot happen: the bin was counted from the same values
            above += sh.pick[1];
            c = ws.in;
            const uint32_t left = span - (b << shift);
            base += b << shift;
            span = (1u << shift) - 1u < left ? (1u << shift) - 1u : left;
            __syncthreads();   // (pick is rewritten)
        }
        if (tid == 0) { ws.base[j] = base; ws.span[j] = span; ws.above[j] = above; ws.c[j] = c; }
    }
    __syncthreads();
    if (arrived) {
        // per unit: what lies above the bin as it is now, inside what it was; what lies inside it
        for (uint32_t x = 0; x < ws.n_own; ++x) {
            const uint32_t u = __builtin_amdgcn_readfirstlane(ws.own[x] * EW + wib);
            if (u >= units) continue;
#pragma unroll 1
            for (int j = 0; j < p.n_cf; ++j) {
                if (ws.mode[j] != MODE_WIDE) continue;
                const uint32_t base = ws.base[j], span = ws.span[j], end = p.st[j].base + p.st[j].span;
                const uint32_t lst = (uint32_t)j * REP + (u & (REP - 1u));
                uint32_t n_above = 0, n_in = 0;
                double sum = 0.0;
                walk(u, [&](uint32_t key, bool live) {
                    const bool from = live && key >= base && key <= end, gt = from && key - base > span, in = from && !gt;
                    const double d = (double)__uint_as_float(key);
                    sum += gt ? d * d : 0.0;
                    n_above += (uint32_t)__popcll(__ballot(gt));
                    const uint64_t m = __ballot(in);
                    n_in += (uint32_t)__popcll(m);
                    if (span == 0u || m == 0ull) return;
                    const int leader = __ffsll((unsigned long long)m) - 1;
                    uint32_t at = 0;
                    if (lane == leader) at = atomicAdd(&p.list_cnt[lst * 32], (uint32_t)__popcll(m));
                    const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)at, leader) + lanes_below(m);
                    if (in && pos < LCAP) {
                        p.list_key[lst * LCAP + pos] = key;
                        p.list_tile[lst * LCAP + pos] = u;
                    }
                });
                sum = wave_sum(sum);
                if (lane == 0) {
                    p.sss[(size_t)u * p.n_cf + j] = sum;
                    if (j == p.commit) { p.tg0[u] = n_above; p.tin[u] = n_in; }
                }
            }
        }
        arrived = wait_for_all(p, ws.n_own, ws.arrived, &p.xq[1], ++waits * n_chunks, tid);
    }
    // (a wait that was given up: gathered_resolve flags the error)
    if (tid < p.n_cf && ws.mode[tid] == MODE_WIDE) ws.mode[tid] = !arrived ? MODE_FAIL : (ws.span[tid] == 0u ? MODE_RESOLVED : MODE_GATHER);
    __syncthreads();
}

// CF j's bin after that, if it was one of those.
__device__ __forceinline__ bool wide_load(const Params& p, int j, int tid, Gathered& g, const WideShared& ws)
{
    if (g.mode != MODE_WIDE) return false;
    gathered_load(p, 0, j, tid, g);
    g.mode = ws.mode[j]; g.base = ws.base[j]; g.span = ws.span[j]; g.above = ws.above[j]; g.c = ws.c[j];
    g.tau = g.base; g.cnt_gt = g.above; g.need = g.k - g.above;   // (if it is one key)
    return g.mode != MODE_FAIL;
}

// Statistics of (segment t, CF j), by one workgroup.
template <int U, bool D>
__device__ __forceinline__ void emit_stats(const Params& p, int t, int j, EmitShared& sh, WideShared& ws)
{
    const int tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    // (a direct call has no refine step to add up the sub-tiles' sums)
    const uint32_t u0 = seg_tile0(p, t) * (D ? SUB : SUB / U), u1 = seg_tile1(p, t) * (D ? SUB : SUB / U);
    const double *ssd = D ? p.ssd : p.ssd_t, *sss = D ? p.ovs : p.sss;
    const bool wide = D && p.status->n_wide != 0;
    Gathered g;
    gathered_load(p, t, j, tid, g);
    // the units' sums, eight units per thread and round, in a fixed order
    double sd = 0.0, sj = 0.0;
    uint32_t kept = 0;   // threshold sparsifier: the entries at or above the threshold
    for (uint32_t v0 = u0 + tid; v0 < u1; v0 += 8 * EWG) {
        double xd[8], xj[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t u = v0 + q * EWG;
            xd[q] = (u < u1) ? ssd[u] : 0.0;
            xj[q] = (u < u1) ? sss[(size_t)u * p.n_cf + j] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) { sd += xd[q]; sj += xj[q]; }
    }
    if (p.bounds_from == BOUNDS_FIXED) {
        for (uint32_t u = u0 + tid; u < u1; u += EWG) kept += p.tg0[u];
        kept = wave_sum(kept);
        if (lane == 0) sh.ws[0][wib] = kept;
    }
    if constexpr (D) {
        if (wide) {
            wide_resolve<U>(p, tid, sh, ws);
            if (wide_load(p, j, tid, g, ws))
                for (uint32_t u = tid; u < p.n_tiles * (SUB / U); u += EWG) sj += p.sss[(size_t)u * p.n_cf + j];
        }
    }
    gathered_resolve(p, tid, g, sh);
    const uint32_t dtau = g.tau - g.base;  // the threshold inside the located bin
    // the entries of the located bin above the threshold (Random-k: and the one at it).  Their order in the gather
    // lists varies from run to run, so their energies are added as integers: every square, exact in binary64, is
    // scaled by a power of two that puts the largest of them below 2^50 and truncated, the sum of up to LCAP of them
    // fits 64 bits and does not depend on the order, and it is off by less than 2^-38 of itself.
    double ebin = 0.0;
    if (g.mode == MODE_GATHER) {
        const auto square = [&](uint32_t d, float val) {
            const bool in = d > dtau || (p.random && d == dtau);
            const double dv = p.random ? (double)val : (double)__uint_as_float(g.base + d);
            return in ? dv * dv : 0.0;
        };
        const uint32_t kmax = g.base + g.span;   // the located bin's largest key
        if (!p.random && kmax < 0x7F800000u) {
            // Top-k keys are magnitudes, and the bin's own bounds say how large a square can get: no look at the
            // entries for the scale, and nothing can be infinite or NaN
            if (kmax != 0u) {
                const double m = (double)__uint_as_float(kmax);
                const int ex = ilogb(m * m);                  // every square is below 2^(ex + 1)
                const double sc = scalbn(1.0, 49 - ex);       // (a power of two: the product is exact)
                uint64_t acc = 0;
                gathered_each(p, tid, g, [&](uint32_t d, uint32_t, float val) { acc += (uint64_t)(square(d, val) * sc); });  // < 2^50 each
                acc = wave_sum(acc);
                if (lane == 0) sh.ured[wib] = acc;
                __syncthreads();
                uint64_t all = 0;
#pragma unroll
                for (int w = 0; w < EW; ++w) all += sh.ured[w];
                ebin = scalbn((double)all, ex - 49);
            }
        } else {
            double mx = 0.0, plain = 0.0;
            bool finite = true;
            gathered_each(p, tid, g, [&](uint32_t d, uint32_t, float val) {
                const double x = square(d, val);
                mx = fmax(mx, x);   // (a NaN square is skipped here and shows in the plain sum)
                plain += x;
                finite = finite && (x <= 1.0e300);
            });
            mx = wave_max(mx);
            if (lane == 0) sh.dred[2][wib] = mx;
            const bool all_finite = __syncthreads_and(finite ? 1 : 0) != 0;
            mx = 0.0;
#pragma unroll
            for (int w = 0; w < EW; ++w) mx = fmax(mx, sh.dred[2][w]);
            __syncthreads();
            if (!all_finite) {
                // an infinite or NaN square: the sum is infinite or NaN in any order
                plain = wave_sum(plain);
                if (lane == 0) sh.dred[2][wib] = plain;
                __syncthreads();
                for (int w = 0; w < EW; ++w) ebin += sh.dred[2][w];
            } else if (mx > 0.0) {
                const int ex = ilogb(mx);                      // 2^ex <= mx < 2^(ex + 1)
                uint64_t acc = 0;
                gathered_each(p, tid, g, [&](uint32_t d, uint32_t, float val) { acc += (uint64_t)scalbn(square(d, val), 49 - ex); });  // < 2^50 each
                acc = wave_sum(acc);
                if (lane == 0) sh.ured[wib] = acc;
                __syncthreads();
                uint64_t all = 0;
#pragma unroll
                for (int w = 0; w < EW; ++w) all += sh.ured[w];
                ebin = scalbn((double)all, ex - 49);
            }
        }
    }
    // every wavefront's sum, then the EW of them in order: the same order in every run
    {
        const double wd = wave_sum(sd), wj = wave_sum(sj);
        if (lane == 0) { sh.dred[0][wib] = wd; sh.dred[1][wib] = wj; }
    }
    __syncthreads();
    if (tid == 0) {
        // fourth statistic: the threshold as a magnitude (Top-k) or as a priority (Random-k)
        const double tauv = p.random ? (double)g.tau : (double)__uint_as_float(g.tau);
        double ss_dense = 0.0, ss_above = 0.0;
        for (int w = 0; w < EW; ++w) { ss_dense += sh.dred[0][w]; ss_above += sh.dred[1][w]; }
        // Top-k: the ties all have magnitude tau; Random-k: the entry at the threshold has been summed
        const double ss_sel = ss_above + ebin + (p.random ? 0.0 : (double)g.need * tauv * tauv);
        double* o = p.out_stats + ((size_t)t * p.n_cf + j) * GRAVAC_STATS_PER_CF;
        o[0] = ss_sel;
        o[1] = ss_dense;
        o[2] = (ss_dense == 0.0) ? 1.0 : ss_sel / ss_dense;
        o[3] = p.bounds_from == BOUNDS_FIXED ? (double)__uint_as_float(p.fixed_key) : tauv;
        if (p.bounds_from == BOUNDS_FIXED) {
            uint32_t n = 0;
            for (int w = 0; w < EW; ++w) n += sh.ws[0][w];
            p.status->count = (int)n;
            *p.out_count = (int64_t)n;
        }
    }
}

constexpr uint32_t EMIT_STAGE = TS / 2;
static_assert(EMIT_STAGE % 256 == 0, "a lane's four pairs are aligned and inside");
// Streamed messages (the forms with S): pairs go through LDS and from there to memory four per lane with non-temporal hints.
// What a kernel leaves in the L2 caches is written back when it ends, and nothing runs meanwhile; the hints have it written as
// it comes, in pieces long enough to fill lines.  Microseconds of a call without and with it, on the same buffers each time and (in
// brackets) on three states in turn, Normal gradients:
//    45 million, CF 10   145.3  143.2  (152.0  146.2)    CF 3    205.2  183.3  (240.4  215.9)    CF 2   223.0  239.4  (255.3  242.7)
//    30 million, CF 10   112.0  110.8  (114.2  112.6)    CF 3    149.6  143.7  (180.4  160.2)    CF 2   162.6  174.1  (185.9  177.9)
//   138 million, CF 10   373.4  358.1  (426.2  405.8)    CF 3    639.8  618.7  (640.4  619.2)    CF 2   700.3  661.6  (701.3  702.7)
// (the VGG16 shape with its two parts, CF 10: 363.7 364.2 (388.5 373.2); a million pairs of 100 million elements 236.9 238.1, hence
// the number below.  As plain stores of 16 bytes it is as it was, and so are hints on stores of a pair per lane: 10 us slower.)
// Where two in five entries or more are selected a wavefront's 64 pairs fill lines by themselves, and a message of a call without a
// scan step is left to the caches, which is slower only where the call before it has filled them with other buffers' results: 45
// million at CF 2 after 512 MB have been read 238.6 260.7, after they have been written 266.9 271.6, Random-k 237.9 263.9 and 273.0
// 278.6.  (66 million and more, with a scan step, are as fast or faster streamed except after a read, 334 363.)
constexpr int64_t STREAM_OUT = 1500000;   // pairs

struct EmitCtx {
    uint32_t tau, take, pz;
    bool put_back;
    bool zero;   // selected entries are removed from the residual (not in a call without commit)
    int64_t pos, lim;
    uint32_t erun;
    int32_t* sidx;     // selected pairs on their way to the message, in LDS: EMIT_STAGE of this wavefront's own ...
    float* sval;
    uint32_t staged;   // ... and their number
    // The first pass has left +0 in the residual of its listed sub-tiles for keys >= pz (not on the full exact route,
    // which has put acc back).  Those entries need no store here if they are selected, and get acc back if they are
    // not, which can only be when the threshold turned out to lie at or above pz.
    __device__ __forceinline__ void set_pz(const Params& p, const SegState& sg, bool single)
    {
        pz = (single || sg.fail == FAIL_FULL) ? NONE : sg.pz;
        put_back = pz != NONE && tau >= pz;
        zero = !p.no_commit;
    }
    __device__ __forceinline__ void set_tau(uint32_t key)
    {
        tau = key;
        put_back = pz != NONE && tau >= pz;
    }
};

// The staged pairs to their place in the message (which starts at any multiple of four bytes).
template <bool GEN>
__device__ __forceinline__ void emit_flush(const Params& p, EmitCtx& x)
{
    const bool single = GEN && p.single;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the wavefront's own LDS writes, read back by other lanes
    const int64_t left = x.lim - x.pos;
    if ((int64_t)x.staged > left) p.status->error = 1;   // cannot happen if the counts are consistent; never write out of range
    const uint32_t n = (int64_t)x.staged > left ? (left > 0 ? (uint32_t)left : 0u) : x.staged;
    // (values and indices one after the other: fewer registers)
#pragma unroll 1
    for (uint32_t i = 4u * (threadIdx.x & 63u); i < n; i += 256) {
        float* to = p.out_val + x.pos + i;
        const v4f b = *(const v4f*)(x.sval + i);
        if (i + 4 <= n) {
            st_stream(b, (v4fu*)to);
        } else {
#pragma unroll
            for (uint32_t e = 0; e < 3; ++e)
                if (i + e < n) to[e] = b[e];
        }
    }
#pragma unroll 1
    for (uint32_t i = 4u * (threadIdx.x & 63u); i < n; i += 256) {
        int32_t* to = p.out_idx + x.pos + i;
        v4i a = *(const v4i*)(x.sidx + i);
        if (single) {
            // positions in the message -> indices in the gradient (a place past the last pair takes the first one's)
            const v4i at = a;
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) a[e] = p.map_idx[i + e < n ? at[e] : at[0]];
            if (p.restore) {
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    if (i + e < n && (uint64_t)(int64_t)a[e] < (uint64_t)p.n_restore) p.restore[a[e]] = 0.0f;
            }
        }
        if (i + 4 <= n) {
            __builtin_nontemporal_store(a, (v4iu*)to);
        } else {
#pragma unroll
            for (uint32_t e = 0; e < 3; ++e)
                if (i + e < n) to[e] = a[e];
        }
    }
    x.pos += x.staged;
    x.staged = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // read before the next pairs overwrite them
}

// One round of up to 64 listed candidates (idx, val), one per lane.
template <bool GEN, bool S>
__device__ __forceinline__ void emit_listed(const Params& p, EmitCtx& x, int32_t idx, float val, bool live)
{
    const bool rnd = GEN && p.random, single = GEN && p.single;
    const uint32_t key = rnd ? priority_of(p.rk_s0, p.rk_s1, (uint32_t)idx) : key_of(val);
    const bool gt = live && key > x.tau, eq = live && key == x.tau;
    const uint64_t me = __ballot(eq);
    bool sel = gt;
    if (me != 0ull) sel = gt || (eq && (x.erun + lanes_below(me)) < x.take);  // (few rounds hold a tie)
    const uint64_t ms = __ballot(sel);
    if constexpr (S) {
        if (x.staged > EMIT_STAGE - 64) emit_flush<GEN>(p, x);
        if (sel) {
            const uint32_t o = x.staged + lanes_below(ms);
            x.sidx[o] = idx;
            x.sval[o] = val;
            if (!single && x.zero && key < x.pz) __builtin_nontemporal_store(0.0f, &p.res[idx]);
        } else if (x.put_back && live && key >= x.pz) {
            p.res[idx] = val;
        }
        x.staged += (uint32_t)__popcll(ms);
        x.erun += (uint32_t)__popcll(me);
        return;
    }
    // the wavefront's pairs go to consecutive places from pos on: a uniform base and a small offset per lane
    const int64_t left = x.lim - x.pos;
    const uint32_t room = left >= 64 ? 64u : (left > 0 ? (uint32_t)left : 0u);
    float* ov = p.out_val + x.pos;
    int32_t* oi = p.out_idx + x.pos;
    if (sel) {
        const uint32_t o = lanes_below(ms);
        if (o < room) {
            ov[o] = val;
            if (!single) {
                oi[o] = idx;
                if (x.zero && key < x.pz) __builtin_nontemporal_store(0.0f, &p.res[idx]);
            } else {
                const int mi = p.map_idx[idx];  // position in the message -> index in the gradient
                oi[o] = mi;
                if (p.restore && (uint64_t)(int64_t)mi < (uint64_t)p.n_restore) p.restore[mi] = 0.0f;
            }
        } else {
            p.status->error = 1;  // cannot happen if the counts are consistent; never write out of range
        }
    } else if (x.put_back && live && key >= x.pz) {
        p.res[idx] = val;
    }
    x.pos += __popcll(ms);
    x.erun += (uint32_t)__popcll(me);
}

// GEN false: compiled for the plain call (Top-k or threshold keys, gradient + residual).
// HEADS (plain call only): the heads of the unit's lists, 32 candidates each of a tile's eight lists, 64 of four, 128 of two, are fetched
// with the kernel's first loads, before the lists' lengths are known; a unit whose lists are no longer than that is emitted from them, a
// lane's four consecutive candidates at a time, one round trip to memory earlier.  As in the refine kernel this
// pays where all tiles' wavefronts are resident at once, and the host picks the form by the number of tiles.
//
// One unit u of segment t, by one wavefront: x holds the threshold, the unit's tie quota and the place of its pairs; cc
// are its sub-tiles' counts, hi4 / hv4 the heads of its lists.
template <bool GEN, bool HEADS, int U, bool S>
__device__ __forceinline__ void emit_unit(const Params& p, int t, uint32_t u, EmitCtx& x, const uint32_t (&cc)[U], const v4i& hi4,
                                          const v4f& hv4, int32_t* sidx, float* sval)
{
    static_assert(!(GEN && HEADS), "the early loads exist in the plain form only");
    const bool rnd = GEN && p.random, single = GEN && p.single;  // (known to be off in the plain form)
    const int lane = threadIdx.x & 63;
    uint32_t dmask = 0;  // bit j: sub-tile j keeps no candidate list
#pragma unroll
    for (int j = 0; j < U; ++j) dmask |= (cc[j] & DENSE_BIT) ? 1u << j : 0u;
    const bool any_dense = dmask != 0u;
    const float* cv = p.cand_val + (size_t)u * (U * TS);
    const int32_t* ci = p.cand_idx + (size_t)u * (U * TS);
    if constexpr (HEADS) {
        constexpr int H = 64 / U;   // lanes per sub-tile
        bool covered = !any_dense;
        uint32_t cj = 0;  // candidates of this lane's sub-tile
#pragma unroll
        for (int j = 0; j < U; ++j) {
            covered = covered && cc[j] <= 4u * H;
            if (lane / H == j) cj = cc[j];
        }
        if (covered) {
            const int32_t ia[4] = {hi4.x, hi4.y, hi4.z, hi4.w};
            const float va[4] = {hv4.x, hv4.y, hv4.z, hv4.w};
            uint32_t key[4];
            bool live[4], sel[4];
            uint32_t n_eq = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                live[e] = 4u * (lane % H) + e < cj;
                key[e] = key_of(va[e]);
                sel[e] = live[e] && key[e] > x.tau;
                n_eq += (live[e] && key[e] == x.tau) ? 1u : 0u;
            }
            if (__ballot(n_eq != 0u) != 0ull) {
                // ties at the threshold: the first x.take of them in index order (lanes are in index order) are selected
                uint32_t rank = wave_scan(n_eq) - n_eq;   // ties in lower lanes
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (live[e] && key[e] == x.tau) { sel[e] = rank < x.take; ++rank; }
                }
            }
            const uint32_t n_sel = (sel[0] ? 1u : 0u) + (sel[1] ? 1u : 0u) + (sel[2] ? 1u : 0u) + (sel[3] ? 1u : 0u);
            uint32_t o = wave_scan(n_sel) - n_sel;       // pairs of lower lanes
            const int64_t left = x.lim - x.pos;
            const uint32_t room = left >= (int64_t)(U * TS) ? (uint32_t)(U * TS) : (left > 0 ? (uint32_t)left : 0u);
            float* ov = p.out_val + x.pos;
            int32_t* oi = p.out_idx + x.pos;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (sel[e]) {
                    if (o < room) {
                        ov[o] = va[e];
                        oi[o] = ia[e];
                        if (x.zero && key[e] < x.pz) p.res[ia[e]] = 0.0f;
                    } else {
                        p.status->error = 1;  // cannot happen if the counts are consistent; never write out of range
                    }
                    ++o;
                } else if (x.put_back && live[e] && key[e] >= x.pz) {
                    p.res[ia[e]] = va[e];
                }
            }
            return;
        }
    }
    UnitLists<U> tl;
    tl.start[0] = 0;
#pragma unroll
    for (int j = 0; j < U; ++j) tl.start[j + 1] = tl.start[j] + (cc[j] & ~DENSE_BIT);
    if (!any_dense && tl.total() < LONG_WALK) {
        // all sub-tiles listed, and shortly: their lists are walked as one, 64 candidates per round.  The loads of
        // the next rounds are issued before this round is worked on (an absent candidate reads slot 0 and is not
        // used), so that a wavefront does not wait a full round trip per round
        const uint32_t cnt = tl.total();
        float vn[4];
        int32_t in[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t q = r * 64 + lane;
            const uint32_t sl = (q < cnt) ? tl.slot(q) : 0u;
            vn[r] = cv[sl];
            in[r] = ci[sl];
        }
        for (uint32_t b0 = 0; b0 < cnt; b0 += 64 * 4) {
            float vq[4];
            int32_t iq[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) { vq[r] = vn[r]; iq[r] = in[r]; }
            if (b0 + 64 * 4 < cnt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t q = b0 + 64 * 4 + r * 64 + lane;
                    const uint32_t sl = (q < cnt) ? tl.slot(q) : 0u;
                    vn[r] = cv[sl];
                    in[r] = ci[sl];
                }
            }
#pragma unroll 1
            for (uint32_t b = b0; b < b0 + 64 * 4 && b < cnt; b += 64) {
                const int32_t idx = pop_front(iq);
                const float val = pop_front(vq);
                emit_listed<GEN, S>(p, x, idx, val, b + lane < cnt);
            }
        }
        if constexpr (S) emit_flush<GEN>(p, x);
        return;
    }
    if (!any_dense) {
        // all sub-tiles listed, at length (a low CF): sub-tile by sub-tile, so that no lane has to search for its
        // candidate's slot, and the first two rounds of every sub-tile are loaded before any is worked on: the
        // wavefront pays one round trip to memory, not one per sub-tile.  Sub-tiles with more than two rounds (CFs below
        // about 7) have the round after the next one on its way while one is worked on (loaded when it is due: 85 instead
        // of 76 us for 2 million elements at CF 3; four rounds at once cost a wavefront per SIMD, 284 instead of 242 us for
        // 60 million at CF 5)
        // (the streamed form, which needs registers for its stores, has the next AHEAD sub-tiles' rounds on their way)
        constexpr int AHEAD = S && U > 4 ? 4 : U;
        float va[2 * AHEAD];
        int32_t ia[2 * AHEAD];
        // (Random-k at CF 10: 151 -> 147 us with non-temporal loads; in the plain form they cost a 25 MB bucket 2 us)
        const auto fetch = [&](int j, int q, float& v, int32_t& i) {
            const size_t at = (size_t)j * TS + q * 64 + lane;
            v = GEN ? __builtin_nontemporal_load(&cv[at]) : cv[at];
            i = GEN ? __builtin_nontemporal_load(&ci[at]) : ci[at];
        };
#pragma unroll
        for (int r = 0; r < 2 * AHEAD; ++r) fetch(r / 2, r & 1, va[r], ia[r]);
#pragma unroll 1
        for (int j = 0; j < U; ++j) {
            uint32_t c = 0;
#pragma unroll
            for (int y = 0; y < U; ++y) c = y == j ? cc[y] : c;
            float v0 = pop_front(va), v1 = pop_front(va);
            int32_t i0 = pop_front(ia), i1 = pop_front(ia);
            if (AHEAD < U && j + AHEAD < U) {
                fetch(j + AHEAD, 0, va[2 * AHEAD - 2], ia[2 * AHEAD - 2]);
                fetch(j + AHEAD, 1, va[2 * AHEAD - 1], ia[2 * AHEAD - 1]);
            }
#pragma unroll 1
            for (uint32_t b = 0; b < c; b += 64) {
                const float val = v0;
                const int32_t idx = i0;
                v0 = v1; i0 = i1;
                if (b + 128 < c) {   // (the round after the next one)
                    const uint32_t q = j * TS + ((b + 128 + lane) & (TS - 1));
                    v1 = cv[q]; i1 = ci[q];
                }
                emit_listed<GEN, S>(p, x, idx, val, b + lane < c);
            }
        }
        if constexpr (S) emit_flush<GEN>(p, x);
        return;
    }
    // sub-tile by sub-tile: a tile with sub-tiles that keep no list
    // (two rows of a sub-tile at a time in LDS, sidx / sval: with room for a whole sub-tile the LDS of a workgroup would
    // limit the kernel to five wavefronts per SIMD, and the listed tiles of the same launch need the occupancy)
    const int64_t tile0 = seg_begin(p, t) + (int64_t)(u - seg_tile0(p, t) * (SUB / U)) * (U * TS);
    v4f nxt[ROWS];  // the rows of the next sub-tile without a list
    {
        const int64_t sn = tile0 + (int64_t)(__ffs((int)dmask) - 1) * TS;
#pragma unroll
        for (int q = 0; q < ROWS; ++q) nxt[q] = ld_stream((const v4fu*)(p.acc + sn + q * ROW + 4 * lane));
    }
    // the first two rounds of the next sub-tile's list, loaded while this one is worked on, whatever they hold
    float vnx[2];
    int32_t inx[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) { vnx[r] = cv[r * 64 + lane]; inx[r] = ci[r * 64 + lane]; }
#pragma unroll 1
    for (int j = 0; j < U; ++j) {
        float vq[2];
        int32_t iq[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) { vq[r] = vnx[r]; iq[r] = inx[r]; }
        if (j + 1 < U) {
#pragma unroll
            for (int r = 0; r < 2; ++r) { vnx[r] = cv[(j + 1) * TS + r * 64 + lane]; inx[r] = ci[(j + 1) * TS + r * 64 + lane]; }
        }
        if (!((dmask >> j) & 1u)) {
            const uint32_t c = p.cand_cnt[(size_t)u * U + j];
#pragma unroll 1
            for (uint32_t b = 0; b < c; b += 64) {
                const float val = vq[0];
                const int32_t idx = iq[0];
                vq[0] = vq[1]; iq[0] = iq[1];
                if (b + 128 < c) {   // (the round after the next one)
                    const uint32_t q = j * TS + ((b + 128 + lane) & (TS - 1));
                    vq[1] = cv[q]; iq[1] = ci[q];
                }
                emit_listed<GEN, S>(p, x, idx, val, b + lane < c);
            }
            continue;
        }
        // a whole sub-tile that kept acc in the residual (or is the message itself, single-source mode):
        // four rows of 256 elements, a lane's four consecutive elements at a time.  Its rows were loaded while the
        // sub-tile before it was worked on; now the next such sub-tile's loads are issued.
        const int64_t s0 = tile0 + (int64_t)j * TS;
        uint32_t staged = 0;  // pairs in LDS so far
        v4f av[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) av[q] = nxt[q];
        {
            const uint32_t later = dmask & ~((2u << j) - 1u);
            if (later != 0u) {
                const int64_t sn = tile0 + (int64_t)(__ffs((int)later) - 1) * TS;
#pragma unroll
                for (int q = 0; q < ROWS; ++q) nxt[q] = ld_stream((const v4fu*)(p.acc + sn + q * ROW + 4 * lane));
            }
        }
#pragma unroll 1
        for (int q = 0; q < ROWS; ++q) {
            const int64_t g = s0 + q * ROW + 4 * lane;
            const v4f row = pop_front(av);
            const float a[4] = {row.x, row.y, row.z, row.w};
            bool gt[4], eq[4], sel[4];
            uint32_t ties_below = 0;   // ties in lower lanes of this row
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t key = rnd ? priority_of(p.rk_s0, p.rk_s1, (uint32_t)(g + e)) : key_of(a[e]);
                gt[e] = key > x.tau;
                eq[e] = key == x.tau;
            }
            uint32_t ties_row = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t m = __ballot(eq[e]);
                ties_below += lanes_below(m);
                ties_row += (uint32_t)__popcll(m);
            }
            uint32_t er = x.erun + ties_below;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sel[e] = gt[e] || (eq[e] && er < x.take);
                er += eq[e] ? 1u : 0u;
            }
            uint32_t pre = 0, tot = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t m = __ballot(sel[e]);
                pre += lanes_below(m);
                tot += (uint32_t)__popcll(m);
            }
            // the selected pairs go to their place in the sub-tile's part of the message, in LDS first
            if constexpr (S) {
                if (x.staged > EMIT_STAGE - ROW) emit_flush<GEN>(p, x);
            }
            uint32_t o = (S ? x.staged : staged) + pre;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (!sel[e]) continue;
                int32_t gi = (int32_t)(g + e);
                if (single && !S) {
                    gi = p.map_idx[g + e];
                    if (p.restore && (uint64_t)(int64_t)gi < (uint64_t)p.n_restore) p.restore[gi] = 0.0f;
                }
                sidx[o] = gi;
                sval[o] = a[e];
                ++o;
            }
            if (!single && x.zero) {
                v4f r;
                r.x = sel[0] ? 0.0f : a[0]; r.y = sel[1] ? 0.0f : a[1];
                r.z = sel[2] ? 0.0f : a[2]; r.w = sel[3] ? 0.0f : a[3];
                st_stream(r, (v4fu*)(p.res + g));   // (non-temporal, as the loads: VGG16 shape at CF 10 408 -> 398 us)
            }
            (S ? x.staged : staged) += tot;
            x.erun += ties_row;
            if (!S && (q & 1)) {
                // ... and from there into the message, 64 consecutive pairs per store
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the wavefront's own LDS writes, read back by other lanes
                if (x.pos + (int64_t)staged > x.lim) p.status->error = 1;  // cannot happen if the counts are consistent
                for (uint32_t i = lane; i < staged; i += 64) {
                    if (x.pos + i < x.lim) {   // never write out of range
                        p.out_idx[x.pos + i] = sidx[i];
                        p.out_val[x.pos + i] = sval[i];
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // read before the next rows overwrite them
                x.pos += staged;
                staged = 0;
            }
        }
    }
    if constexpr (S) emit_flush<GEN>(p, x);
}

// After the scan step.
template <bool GEN, bool S>
__global__ __launch_bounds__(LWG) void emit_kernel(Params p)
{
    __shared__ __attribute__((aligned(16))) int32_t stage_idx[LWAVES][EMIT_STAGE];   // half a sub-tile's part of the message, per wavefront
    __shared__ __attribute__((aligned(16))) float stage_val[LWAVES][EMIT_STAGE];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
    const uint32_t u = __builtin_amdgcn_readfirstlane(blockIdx.x * LWAVES + wib);
    if (u >= p.n_tiles) return;
    uint32_t cc[SUB];
#pragma unroll
    for (int j = 0; j < SUB; ++j) cc[j] = p.cand_cnt[(size_t)u * SUB + j];
    const int t = tile_seg(p, u);
    EmitCtx x;
    x.take = p.ttake[u];
    x.tau = p.st[(size_t)t * p.n_cf + p.commit].tau;
    x.set_pz(p, p.seg[t], GEN && p.single);
    if (p.bounds_from == BOUNDS_FIXED && (int64_t)p.status->count > p.total_out) {
        // threshold sparsifier, more entries kept than the caller's buffers hold: nothing is emitted and nothing removed.
        // The listed sub-tiles get back the values the pass replaced by +0; the others kept acc.
        for (int j = 0; j < SUB; ++j) put_back_subtile(p, u * SUB + j, x.pz, lane);
        return;
    }
    if (p.tsel[u] == 0 && !x.put_back) return;
    const int64_t seg_out = seg_koff(p, t);
    x.lim = seg_out + (int64_t)seg_k(p, t, p.commit);  // end of this segment's message
    x.pos = seg_out + (int64_t)p.toff[u];
    x.erun = 0;
    x.sidx = stage_idx[wib]; x.sval = stage_val[wib]; x.staged = 0;
    emit_unit<GEN, false, SUB, S>(p, t, u, x, cc, v4i{0, 0, 0, 0}, v4f{0.0f, 0.0f, 0.0f, 0.0f}, stage_idx[wib], stage_val[wib]);
}

// Without a scan step.
template <bool GEN, int U, bool D, bool S>
__global__ __launch_bounds__(EWG) __attribute__((amdgpu_waves_per_eu(D ? 4 : 6, 8))) void resolve_emit_kernel(Params p)
{
    constexpr bool HEADS = !GEN;
    constexpr int H = 64 / U;   // lanes per sub-tile's list
    __shared__ EmitShared sh;
    __shared__ WideShared ws;   // (D)
    __shared__ __attribute__((aligned(16))) int32_t stage_idx[EW][TS / 2];   // half a sub-tile's part of the message, per wavefront
    __shared__ __attribute__((aligned(16))) float stage_val[EW][TS / 2];     // (before that: the heads of the tile's lists)
    const int tid = threadIdx.x, lane = tid & 63, wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t n_stats = (uint32_t)p.n_seg * p.n_cf;
    if (blockIdx.x < n_stats) {
        const int t = (int)(blockIdx.x / (uint32_t)p.n_cf);
        if (!seg_small(p, t)) emit_stats<U, D>(p, t, (int)(blockIdx.x - (uint32_t)t * p.n_cf), sh, ws);
        return;
    }
    // ---- this workgroup's tiles [ub, ue) of segment t, a wavefront each
    const uint32_t w = blockIdx.x - n_stats;
    const int t = is_flat(p) ? 0 : (int)p.wseg[w];
    const uint32_t u0 = seg_tile0(p, t) * (SUB / U), u1 = seg_tile1(p, t) * (SUB / U);
    const uint32_t ub = u0 + (is_flat(p) ? w : w - p.segs[t].wg0) * EW, ue = ub + EW < u1 ? ub + EW : u1;
    // ---- loads that depend on nothing else, in flight together
    v4i hi4 = {0, 0, 0, 0};
    v4f hv4 = {0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t cc[U];
    {
        const uint32_t u = ub + wib < ue ? ub + wib : ub;
        if constexpr (HEADS) {
            // lane l: candidates 4 (l % H) .. + 3 of sub-tile l / H (16-byte aligned: a sub-tile's slots start at a multiple of TS)
            const size_t at = (size_t)u * (U * TS) + (size_t)(lane / H) * TS + 4u * (lane % H);
            hi4 = *(const v4i*)(p.cand_idx + at);
            hv4 = *(const v4f*)(p.cand_val + at);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) cc[j] = p.cand_cnt[(size_t)u * U + j];
    }
    if (tid < EW) {
        const bool mine = ub + tid < ue;
        uint32_t n_above = 0, n_in = 0;
        if (mine && D) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const uint32_t v = (ub + tid) * U + i;
                n_above += p.ovn[(size_t)v * p.n_cf + p.commit];
                n_in += p.brk_cnt[v] >> ZERO_SHIFT;
            }
        } else if (mine) {
            n_above = p.tg0[ub + tid];
            n_in = p.tin[ub + tid];
        }
        sh.tg[tid] = n_above;
        sh.te[tid] = n_in;
        sh.fg[tid] = 0;
        sh.fe[tid] = 0;
    }
    // what lies before the workgroup's tiles in the segment: whole groups of CTILES tiles, and single tiles at both ends
    // (a direct call: single sub-tiles; what a bin that is resolved has in them are zeros)
    uint32_t pg = 0, pe = 0;
    if constexpr (D) {
        for (uint32_t v = tid; v < ub * U; v += EWG) { pg += p.ovn[(size_t)v * p.n_cf + p.commit]; pe += p.brk_cnt[v] >> ZERO_SHIFT; }
    } else {
        const uint32_t g0 = (u0 + CTILES - 1u) / CTILES, g1 = ub / CTILES;   // whole groups, if g0 < g1
        const uint32_t head = g0 * CTILES < ub ? g0 * CTILES : ub, tail = g1 > g0 ? g1 * CTILES : head;
        for (uint32_t i = g0 + tid; i < g1; i += EWG) { const uint64_t v = p.csum[(size_t)i * 8]; pg += (uint32_t)(v >> 32); pe += (uint32_t)v; }
        if (u0 + tid < head) { pg += p.tg0[u0 + tid]; pe += p.tin[u0 + tid]; }
        if (tail + tid < ub) { pg += p.tg0[tail + tid]; pe += p.tin[tail + tid]; }
    }
    const SegState sg = p.seg[t];
    const bool wide = D && p.status->n_wide != 0;
    Gathered g;
    gathered_load(p, t, p.commit, tid, g);
    if constexpr (HEADS) {   // (out of the registers while the threshold is resolved)
        *(v4i*)&stage_idx[wib][4 * lane] = hi4;
        *(v4f*)&stage_val[wib][4 * lane] = hv4;
    }
    EmitCtx x;
    x.tau = 0;
    x.set_pz(p, sg, GEN && p.single);
    if (p.bounds_from == BOUNDS_FIXED) {
        uint32_t n = 0;
        for (uint32_t i = tid; i < (p.n_tiles * (SUB / U) + CTILES - 1u) / CTILES; i += EWG) n += (uint32_t)(p.csum[(size_t)i * 8] >> 32);
        n = wave_sum(n);
        if (lane == 0) sh.ws[2][wib] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int i = 0; i < EW; ++i) n += sh.ws[2][i];
        if ((int64_t)n > p.total_out) {   // (as in emit_kernel)
            for (uint32_t v = ub * U + wib; v < ue * U; v += EW) put_back_subtile(p, v, x.pz, lane);
            return;
        }
    }
    if constexpr (D) {
        if (wide) {
            wide_resolve<U>(p, tid, sh, ws);
            if (wide_load(p, p.commit, tid, g, ws)) {
                // what the units have above and inside the bin as it is now
                if (tid < EW && ub + tid < ue) { sh.tg[tid] += p.tg0[ub + tid]; sh.te[tid] = p.tin[ub + tid]; }
                pe = 0;
                for (uint32_t u = tid; u < ub; u += EWG) { pg += p.tg0[u]; pe += p.tin[u]; }
            }
        }
    }
    gathered_resolve(p, tid, g, sh);
    const uint32_t dtau = g.tau - g.base;  // the threshold inside the located bin
    // ---- the gathered entries above and at the threshold, by tile.  Entries equal to tau: those inside a located bin
    // that is one key wide, else the gathered ones
    const bool one_key = g.mode == MODE_RESOLVED;
    if (!one_key) pe = 0;
    if (g.mode == MODE_GATHER) {
        gathered_each(p, tid, g, [&](uint32_t d, uint32_t tile, float) {
            if (d < dtau) return;
            const bool gt = d > dtau;
            if (tile < ub) { if (gt) ++pg; else ++pe; }
            else if (tile < ue) atomicAdd(gt ? &sh.fg[tile - ub] : &sh.fe[tile - ub], 1u);
        });
    }
    pg = wave_sum(pg);
    pe = wave_sum(pe);
    if (lane == 0) { sh.ws[0][wib] = pg; sh.ws[1][wib] = pe; }
    __syncthreads();
    if (ub + wib >= ue) return;
    // ---- this wavefront's tile: pairs before it, ties before it, its own
    uint32_t run_g = 0, run_e = 0, tg = 0, te = 0;
#pragma unroll
    for (int i = 0; i < EW; ++i) {
        run_g += sh.ws[0][i];
        run_e += sh.ws[1][i];
        const uint32_t gi = sh.tg[i] + sh.fg[i], ei = one_key ? sh.te[i] : sh.fe[i];
        if (i < wib) { run_g += gi; run_e += ei; }
        if (i == wib) { tg = gi; te = ei; }
    }
    const uint32_t ties_before = run_e < g.need ? run_e : g.need;   // ties selected in earlier tiles
    const uint32_t left = g.need - ties_before;
    x.set_tau(__builtin_amdgcn_readfirstlane(g.tau));
    x.take = __builtin_amdgcn_readfirstlane(left < te ? left : te);
    if (__builtin_amdgcn_readfirstlane(tg) + x.take == 0 && !x.put_back) return;
    const int64_t seg_out = seg_koff(p, t);
    x.lim = seg_out + (int64_t)seg_k(p, t, p.commit);  // end of this segment's message
    x.pos = seg_out + (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane(run_g + ties_before);
    x.erun = 0;
    x.sidx = stage_idx[wib]; x.sval = stage_val[wib]; x.staged = 0;
    if constexpr (HEADS) {
        hi4 = *(const v4i*)&stage_idx[wib][4 * lane];
        hv4 = *(const v4f*)&stage_val[wib][4 * lane];
    }
    emit_unit<GEN, HEADS, U, S>(p, t, ub + wib, x, cc, hi4, hv4, stage_idx[wib], stage_val[wib]);
}

// ---------------------------------------------------------------------------------------------
// decompression: dense_out[idx] += val, workers in order.  A workgroup owns one tile of DTILE floats
// of dense_out at a time (tiles are dealt round-robin over a fixed number of workgroups).  A tile
// that lies outside every message's index range is skipped without touching memory.  Otherwise the
// tile's range in every worker's index-sorted message is found by a 32-way search (32 threads per
// worker, both ends at once, 8 workers at a time); if any message touches the tile it is loaded
// into LDS, the pairs are applied worker by worker (indices within one worker are unique, so plain
// LDS adds suffice) and it is written back.
// ---------------------------------------------------------------------------------------------
constexpr int DTILE = 8192;  // floats of dense_out per tile (32 KiB of LDS)
constexpr int DMAXW = 64;    // workers per launch
constexpr int DGROUP = 8;    // workers searched at a time
constexpr int DBATCH = 4;    // pairs per thread and batch
#ifndef GRAVAC_DSPARSE
#define GRAVAC_DSPARSE 512
#endif
constexpr uint32_t DSPARSE = GRAVAC_DSPARSE;   // a tile with at most this many pairs is updated entry by entry
constexpr int DSLOTS = (DSPARSE + 255) / 256;  // pairs per thread of such a tile

struct WorkerOffsets {
    int64_t at[DMAXW + 1];
};

// Both first positions l, h in [a, b) of the ascending array idx with idx[l] >= x0 and idx[h] >= x1
// (x0 <= x1; b if none).  Run by the 32 lanes of one half of a wavefront together; `half` = 0 or 1
// says which half, j = lane within the half.  Each round probes both brackets at once.
__device__ __forceinline__ void lower_bounds_32(const int32_t* idx, int64_t a, int64_t b, int64_t x0, int64_t x1, int half,
                                                int j, int64_t& l, int64_t& h)
{
    int64_t a0 = a, b0 = b, a1 = a, b1 = b;
    bool done0 = false, done1 = false;
    while (!(done0 && done1)) {
        const int64_t n0 = b0 - a0, n1 = b1 - a1;
        const int64_t st0 = n0 > 32 ? (n0 + 31) / 32 : 1, st1 = n1 > 32 ? (n1 + 31) / 32 : 1;
        const int64_t p0 = a0 + (int64_t)j * st0, p1 = a1 + (int64_t)j * st1;
        const bool q0 = !done0 && p0 < b0, q1 = !done1 && p1 < b1;
        const int32_t v0 = q0 ? idx[p0] : 0, v1 = q1 ? idx[p1] : 0;
        const uint32_t c0 = (uint32_t)__popc((uint32_t)(__ballot(q0 && (int64_t)v0 < x0) >> (32 * half)));
        const uint32_t c1 = (uint32_t)__popc((uint32_t)(__ballot(q1 && (int64_t)v1 < x1) >> (32 * half)));
        if (!done0) {
            if (n0 <= 32) { a0 += c0; done0 = true; }            // every position was probed
            else if (c0 == 0) { done0 = true; }                  // idx[a0] >= x0
            else { const int64_t e = a0 + (int64_t)c0 * st0; a0 += (int64_t)(c0 - 1) * st0 + 1; b0 = e < b0 ? e : b0; }
        }
        if (!done1) {
            if (n1 <= 32) { a1 += c1; done1 = true; }
            else if (c1 == 0) { done1 = true; }
            else { const int64_t e = a1 + (int64_t)c1 * st1; a1 += (int64_t)(c1 - 1) * st1 + 1; b1 = e < b1 ? e : b1; }
        }
    }
    l = a0;
    h = a1;
}

// How whole tiles are moved: six of their eight rows of 1024 floats are read with non-temporal hints and seven are written
// with them; in a buffer between PLAIN_FROM and PLAIN_BYTES none is written with them.  Microseconds, eight messages of CF 100 unless
// said, with a workspace; rows hinted (read, written):  0, 0    8, 0    8, 8    8, 6    6, 7
//   178 MB, three buffers in turn                        85.5    82.4    73.6    70.7    70.2
//   178 MB, the same buffer again                        67.2    68.5    73.4    69.1    67.9
//   178 MB, the buffer just cleared                      69.4    69.8    81.8*   68.6    68.6
//   178 MB, caches flushed                               93.5    90.8    83.3    85.3    86.7
//   178 MB, caches flushed, the buffer cleared           79.1    72.0    92.4    79.3    72.4
//   553 MB                                              255     246     225     232     198
//   80 MB, the same buffer again                         33.7    34.2    36.0    35.9    35.9
//   VGG16 shape at CF 1000, 59 of 553 MB, in the step    31.6    31.6    34.4    33.9    33.8
//   ... the step with it, one buffer / three in turn    344/360 346/360 348/348 348/350 348/349
// (*: 68.3 until something else has filled the 256 MB last-level cache once.)  What the hints gain is the cache's evictions
// of dirty lines, which a later kernel pays for unless the same lines are written again soon; with every row hinted a
// buffer that would fit is never taken in again, not even by a clear.  In the last two rows the plain stores only move the
// time from the decompression to the pass over the gradient, as soon as anything else gets into the cache.
// Without a workspace all rows are hinted, read and written, or in a buffer of that size only read (178 MB, three in turn, the
// same again, cleared, flushed: 0, 0: 87, 76, 79, 108; 8, 0: 83, 76, 79, 98; 6, 7: 79, 82, 77, 100; 8, 8: 78, 82, 77, 95).
// A buffer of up to 32 MB fits the eight L2 caches, which would write its lines back when the kernel ends: 16 MB, CF 20,
// in turn 19.3 (6, 0), 17.8 (6, 7); 48 MB 23.1 and 24.6, 64 MB 28.4 and 30.1, 80 MB 36.3 and 35.7, 96 MB 44.7 and 42.0,
// there the same buffer again 40.7 and 42.0.
constexpr int64_t PLAIN_FROM = 32ll << 20, PLAIN_BYTES = 96ll << 20;

template <int NT>  // rows read with hints
__device__ __forceinline__ void load_tile(const float* from, float* acc, int tid)
{
    // (all loads of a thread in flight together)
    v4f tv[DTILE / 1024];
#pragma unroll
    for (int r = 0; r < NT; ++r) tv[r] = ld_stream((const v4fu*)(from + r * 1024 + tid * 4));
#pragma unroll
    for (int r = NT; r < DTILE / 1024; ++r) tv[r] = *(const v4f*)(from + r * 1024 + tid * 4);
#pragma unroll
    for (int r = 0; r < DTILE / 1024; ++r) *(v4f*)(acc + r * 1024 + tid * 4) = tv[r];
}

template <int NT>  // rows written with hints
__device__ __forceinline__ void store_tile(const float* acc, float* to, int tid)
{
#pragma unroll
    for (int r = 0; r < NT; ++r) st_stream(*(const v4f*)(acc + r * 1024 + tid * 4), (v4fu*)(to + r * 1024 + tid * 4));
#pragma unroll
    for (int r = NT; r < DTILE / 1024; ++r) *(v4f*)(to + r * 1024 + tid * 4) = *(const v4f*)(acc + r * 1024 + tid * 4);
}

template <int NT>  // rows of a whole tile written with non-temporal hints
__global__ __launch_bounds__(256) void decompress_kernel(const int32_t* __restrict__ idx, const float* __restrict__ val,
                                                         WorkerOffsets wo, int W, int64_t n, float* dense, float alpha)
{
    __shared__ __attribute__((aligned(16))) float acc[DTILE];
    __shared__ int64_t lo[DGROUP], hi[DGROUP];
    __shared__ uint32_t pre[DGROUP + 1];
    __shared__ int32_t first[DMAXW], last[DMAXW];   // smallest and largest index of every worker's message
    const int tid = threadIdx.x;
    const bool vec = (((uintptr_t)dense) & 15) == 0;  // float4 access needs a 16-byte aligned buffer
    if (tid < W) {
        const int64_t a = wo.at[tid], b = wo.at[tid + 1];
        first[tid] = (b > a) ? idx[a] : 0x7FFFFFFF;
        last[tid] = (b > a) ? idx[b - 1] : -1;
    }
    __syncthreads();
    const int64_t ntile = (n + DTILE - 1) / DTILE;
    for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int64_t base = tile * DTILE;
        const int len = (int)((n - base < DTILE) ? n - base : DTILE);
        bool loaded = false;
        for (int w0 = 0; w0 < W; w0 += DGROUP) {
            const int wn = (W - w0 < DGROUP) ? W - w0 : DGROUP;
            // can any message of this group touch the tile at all?
            bool maybe = false;
            for (int w = 0; w < wn; ++w)
                maybe |= ((int64_t)first[w0 + w] < base + len) && ((int64_t)last[w0 + w] >= base);
            if (!maybe) continue;
            __syncthreads();  // lo / hi / pre of the previous group or tile are no longer read
            {
                const int w = tid >> 5, j = tid & 31, half = (tid >> 5) & 1;
                // 32 threads per worker; absent workers search an empty range
                const int64_t a = (w < wn) ? wo.at[w0 + w] : 0, b = (w < wn) ? wo.at[w0 + w + 1] : 0;
                int64_t l, h;
                lower_bounds_32(idx, a, b, base, base + len, half, j, l, h);
                if (j == 0 && w < wn) { lo[w] = l; hi[w] = h; }
            }
            __syncthreads();
            if (tid == 0) {
                uint32_t s = 0;
                for (int w = 0; w < DGROUP; ++w) {
                    pre[w] = s;
                    if (w < wn) s += (uint32_t)(hi[w] - lo[w]);
                }
                pre[DGROUP] = s;
            }
            __syncthreads();
            const uint32_t total = pre[DGROUP];
            if (total == 0) continue;  // no message of this group touches the tile
            if (W <= DGROUP && total <= DSPARSE) {
                // few pairs, and this group is all there is: only the entries they name are read and written back (as in
                // the kernel that works from tile boundaries; they still go through the tile buffer, worker by worker)
                int pj[DSLOTS], pw[DSLOTS];
                float pv[DSLOTS], dv[DSLOTS];
                int64_t at[DSLOTS];
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q) {
                    const uint32_t slot = q * 256 + tid;
                    const uint32_t sc = slot < total ? slot : total - 1;
                    int w = 0;
#pragma unroll
                    for (int x = 1; x < DGROUP; ++x) w += (sc >= pre[x]);
                    at[q] = lo[w] + (int64_t)(sc - pre[w]);
                    pw[q] = slot < total ? w : -1;
                }
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q) pj[q] = idx[at[q]];
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q) pv[q] = val[at[q]];
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q) {
                    const int64_t j = (int64_t)pj[q] - base;
                    if (j < 0 || j >= len) pw[q] = -1;   // an index outside the tile (malformed message) is ignored
                    pj[q] = (int)(j < 0 || j >= len ? 0 : j);
                }
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q) dv[q] = pw[q] >= 0 ? dense[base + pj[q]] : 0.0f;
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q)
                    if (pw[q] >= 0) acc[pj[q]] = dv[q];  // the same value from every pair of that entry
                __syncthreads();
                for (int w = 0; w < wn; ++w) {
                    if (pre[w + 1] == pre[w]) continue;
#pragma unroll
                    for (int q = 0; q < DSLOTS; ++q)
                        if (pw[q] == w) acc[pj[q]] = __fadd_rn(acc[pj[q]], __fmul_rn(alpha, pv[q]));
                    __syncthreads();
                }
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q)
                    if (pw[q] >= 0) dense[base + pj[q]] = acc[pj[q]];
                continue;   // (nothing was loaded whole: nothing is written back; the next tile starts with a barrier)
            }
            if (!loaded) {
                if (vec && len == DTILE) {
                    load_tile<DTILE / 1024>(dense + base, acc, tid);
                } else {
                    for (int i = tid * 4; i < len; i += 256 * 4) {
                        if (vec && i + 4 <= len) {
                            const v4f v = *(const v4f*)(dense + base + i);
                            acc[i] = v.x; acc[i + 1] = v.y; acc[i + 2] = v.z; acc[i + 3] = v.w;
                        } else {
                            for (int e = 0; e < 4 && i + e < len; ++e) acc[i + e] = dense[base + i + e];
                        }
                    }
                }
                loaded = true;
            }
            // the group's pairs, worker-major, DBATCH per thread and batch; all loads of a batch in flight together
            for (uint32_t s0 = 0; s0 < total; s0 += 256 * DBATCH) {
                int pj[DBATCH], pw[DBATCH];
                float pv[DBATCH];
                int64_t at[DBATCH];
                // where the pairs lie (a slot past the last pair takes the last pair's place and is not applied:
                // total >= 1 here), then all loads without branches around them, in flight together
#pragma unroll
                for (int q = 0; q < DBATCH; ++q) {
                    const uint32_t slot = s0 + q * 256 + tid;
                    const uint32_t sc = slot < total ? slot : total - 1;
                    int w = 0;
#pragma unroll
                    for (int x = 1; x < DGROUP; ++x) w += (sc >= pre[x]);
                    at[q] = lo[w] + (int64_t)(sc - pre[w]);
                    pw[q] = slot < total ? w : -1;
                }
#pragma unroll
                for (int q = 0; q < DBATCH; ++q) pj[q] = idx[at[q]];
#pragma unroll
                for (int q = 0; q < DBATCH; ++q) pv[q] = val[at[q]];
#pragma unroll
                for (int q = 0; q < DBATCH; ++q) {
                    const int64_t j = (int64_t)pj[q] - base;
                    if (j < 0 || j >= len) pw[q] = -1;   // an index outside the tile (malformed message) is ignored
                    pj[q] = (int)(j < 0 || j >= len ? 0 : j);
                }
                // workers present in this batch: from the worker of its first slot to that of its last
                const uint32_t end = (s0 + 256 * DBATCH < total ? s0 + 256 * DBATCH : total) - 1;
                int wmin = 0, wmax = 0;
#pragma unroll
                for (int x = 1; x < DGROUP; ++x) { wmin += (s0 >= pre[x]); wmax += (end >= pre[x]); }
                __syncthreads();  // tile loaded / previous batch applied
                for (int w = wmin; w <= wmax; ++w) {
#pragma unroll
                    for (int q = 0; q < DBATCH; ++q)
                        if (pw[q] == w) acc[pj[q]] = __fadd_rn(acc[pj[q]], __fmul_rn(alpha, pv[q]));
                    __syncthreads();
                }
            }
        }
        if (loaded) {
            __syncthreads();
            if (vec && len == DTILE) {
                store_tile<NT>(acc, dense + base, tid);
            } else {
                for (int i = tid * 4; i < len; i += 256 * 4) {
                    if (vec && i + 4 <= len) {
                        v4f v;
                        v.x = acc[i]; v.y = acc[i + 1]; v.z = acc[i + 2]; v.w = acc[i + 3];
                        *(v4f*)(dense + base + i) = v;
                    } else {
                        for (int e = 0; e < 4 && i + e < len; ++e) dense[base + i + e] = acc[i + e];
                    }
                }
            }
            __syncthreads();  // the tile buffer is free again
        }
    }
}

// ---------------------------------------------------------------------------------------------
// decompression with a workspace: the tile boundaries of every message are computed once, by one thread
// per pair, instead of being searched for by every tile.
//   bounds[w][t], tile(first index of w) < t <= tile(last index of w): number of pairs of worker w with index
//   below t * DTILE (indices below 0 count as tile 0, indices from ntile * DTILE on as past the last tile).
//   Tile t's pairs of worker w are [bounds[w][t], bounds[w][t + 1]) of its message, where the lower end is 0
//   for the tile of the message's first index and the upper end the message's length for the tile of its last
//   index; entries outside that range are never written and never read.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int64_t tile_of_index(int32_t x, int64_t ntile)
{
    if (x < 0) return 0;
    const int64_t t = (int64_t)x / DTILE;
    return t < ntile ? t : ntile;
}

// grid (pair blocks, workers).  Pair j > 0 of a message starts the tiles (tile of pair j - 1, tile of pair j].  A
// wavefront takes BP consecutive rows of 64 pairs, all their loads in flight at once.  A lane with up to BGAP tiles to
// write does it itself, longer runs (gaps in the message) are written by the whole wavefront.
constexpr int BGAP = 8;
// Four rows from this many pairs of a call on, one row below (whole calls, one row and four): 3.6 million pairs 76.5 and
// 73.4 us, 1.6 million 18.4 and 17.5, 0.8 million 14.2 and 14.3, 0.32 million 15.7 and 16.2, 84,000 14.5 and 15.0 (the
// chains are longer and the code is four times as much, on a chip that is not full).
constexpr int64_t BROWS_PAIRS = 1 << 19;

template <int BP>
__global__ __launch_bounds__(256) void bounds_kernel(const int32_t* __restrict__ idx, WorkerOffsets wo, int64_t ntile,
                                                     uint32_t* __restrict__ bounds)
{
    const int w = blockIdx.y, lane = threadIdx.x & 63;
    const int64_t a = wo.at[w], cnt = wo.at[w + 1] - a;
    uint32_t* bw = bounds + (size_t)w * (size_t)(ntile + 1);
    const int64_t j0 = ((int64_t)blockIdx.x * 256 + (threadIdx.x & ~63)) * BP;  // first pair of this wavefront
    if (j0 >= cnt) return;
    int32_t x[BP];
#pragma unroll
    for (int q = 0; q < BP; ++q) {
        const int64_t j = j0 + q * 64 + lane;
        x[q] = idx[a + (j < cnt ? j : cnt - 1)];
    }
    int32_t last = j0 > 0 ? idx[a + j0 - 1] : 0;   // the pair before the row
#pragma unroll
    for (int q = 0; q < BP; ++q) {
        const int64_t j = j0 + q * 64 + lane;
        int32_t prev = __shfl_up(x[q], 1, 64);
        if (lane == 0) prev = last;
        last = __builtin_amdgcn_readlane(x[q], 63);
        const bool live = j > 0 && j < cnt;
        int64_t t_prev = 0, t_cur = 0;  // this lane writes bw[t] = j for t in (t_prev, t_cur]
        if (live) {
            t_cur = tile_of_index(x[q], ntile);
            t_prev = tile_of_index(prev, ntile);
        }
        const int64_t gap = t_cur - t_prev;  // <= 0 where the indices do not ascend: nothing is written
        if (live && gap > 0 && gap <= BGAP)
            for (int64_t t = t_prev + 1; t <= t_cur; ++t) bw[t] = (uint32_t)j;
        uint64_t big = __ballot(live && gap > BGAP);
        while (big) {
            const int src = __ffsll((unsigned long long)big) - 1;
            big &= big - 1;
            const int64_t tp = __shfl(t_prev, src, 64), tc = __shfl(t_cur, src, 64);
            const uint32_t v = (uint32_t)(j0 + q * 64 + src);
            for (int64_t t = tp + 1 + lane; t <= tc; t += 64) bw[t] = v;
        }
    }
}

constexpr int DCHUNK = 32;  // tiles whose boundaries a workgroup fetches in one round of loads
constexpr int DENT = 768;   // (tile, worker) entries of such a chunk

// The tile's pairs in worker-major order, N per thread: place inside the tile, value and worker (-1: none, or an index
// outside the tile, which a malformed message may have).  Slots past the last pair take the last pair's place.
template <int N>
__device__ __forceinline__ void tile_pairs(const int32_t* __restrict__ idx, const float* __restrict__ val, const uint32_t* spre,
                                           const int64_t* wat, const uint32_t* lo, uint32_t tot, int64_t base, int len, int tid,
                                           int (&pj)[N], float (&pv)[N], int (&pw)[N])
{
    int64_t at[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t slot = q * 256 + tid;
        const uint32_t sc = slot < tot ? slot : tot - 1;
        int w = 0;
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1)
            if (spre[w + step] <= sc) w += step;   // spre[64] = tot > sc: w stays below 64
        at[q] = wat[w] + (int64_t)lo[w] + (int64_t)(sc - spre[w]);
        pw[q] = slot < tot ? w : -1;
    }
#pragma unroll
    for (int q = 0; q < N; ++q) pj[q] = idx[at[q]];
#pragma unroll
    for (int q = 0; q < N; ++q) pv[q] = val[at[q]];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int64_t j = (int64_t)pj[q] - base;
        if (j < 0 || j >= len) pw[q] = -1;
        pj[q] = (int)(j < 0 || j >= len ? 0 : j);
    }
}

// (Moving only the named 64-byte lines of a whole tile, seven in ten with eight messages of CF 100, was no faster: 128
// bytes is what the memory moves.)
// A workgroup takes the tiles blockIdx.x, blockIdx.x + gridDim.x, ...  It first fetches, for a chunk of its
// tiles at once, every worker's boundaries (one round of independent loads instead of one dependent round per
// tile) and then walks over the chunk's tiles; a tile no message has a pair in costs no further memory access.
template <int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void decompress_ws_kernel(const int32_t* __restrict__ idx, const float* __restrict__ val,
                                                            WorkerOffsets wo, int W, int64_t n, float* dense,
                                                            const uint32_t* __restrict__ bounds, float alpha)
{
    __shared__ __attribute__((aligned(16))) float acc[DTILE];
    __shared__ uint32_t blo[DENT], bcnt[DENT];      // first pair and number of pairs, per (tile of the chunk, worker)
    __shared__ uint32_t btot[DCHUNK];               // pairs of all workers, per tile of the chunk
    __shared__ uint32_t bwrk[DCHUNK];               // ... the number of those workers (high half) and the sum of their numbers
    __shared__ uint32_t tpre[DCHUNK + 1];           // pairs of the chunk's tiles of one worker before each
    __shared__ uint32_t spre[DMAXW + 1];            // a sparse tile's pairs before worker w, in worker-major order
    __shared__ int64_t wat[DMAXW + 1];              // start of every worker's message
    __shared__ int32_t first[DMAXW], last[DMAXW];   // smallest and largest index of every worker's message
    const int tid = threadIdx.x;
    const bool vec = (((uintptr_t)dense) & 15) == 0;  // float4 access needs a 16-byte aligned buffer
    if (tid <= DMAXW) wat[tid] = wo.at[tid];
    if (tid < W) {
        const int64_t a = wo.at[tid], b = wo.at[tid + 1];
        first[tid] = (b > a) ? idx[a] : 0x7FFFFFFF;
        last[tid] = (b > a) ? idx[b - 1] : -1;
    }
    const int64_t ntile = (n + DTILE - 1) / DTILE;
    const int Wp = (W + DGROUP - 1) / DGROUP * DGROUP;            // workers, padded to whole groups
    const int tc = DENT / Wp < DCHUNK ? DENT / Wp : DCHUNK;       // tiles per chunk (>= 12: Wp <= 64)
    for (int64_t c0 = blockIdx.x; c0 < ntile; c0 += (int64_t)tc * gridDim.x) {
        __syncthreads();  // first / last / wat are written; the previous chunk's entries are no longer read
        if (tid < DCHUNK) { btot[tid] = 0; bwrk[tid] = 0; }
        __syncthreads();
        for (int e = tid; e < tc * Wp; e += 256) {
            const int i = e / Wp, w = e - i * Wp;
            const int64_t tile = c0 + (int64_t)i * gridDim.x;
            uint32_t l = 0, c = 0;
            if (w < W && tile < ntile) {
                const int64_t base = tile * DTILE, end = (n - base < DTILE) ? n : base + DTILE;
                if ((int64_t)first[w] < end && (int64_t)last[w] >= base) {
                    const uint32_t* bw = bounds + (size_t)w * (size_t)(ntile + 1) + tile;
                    const uint32_t cw = (uint32_t)(wat[w + 1] - wat[w]);
                    uint32_t h = cw;
                    if (tile > tile_of_index(first[w], ntile)) l = bw[0];
                    if (tile < tile_of_index(last[w], ntile)) h = bw[1];
                    // clamped to the message, so that no read can leave it even if the indices were not ascending
                    l = l < cw ? l : cw;
                    h = h < l ? l : (h < cw ? h : cw);
                    c = h - l;
                }
            }
            blo[e] = l;
            bcnt[e] = c;
            if (c) { atomicAdd(&btot[i], c); atomicAdd(&bwrk[i], 0x10000u + (uint32_t)w); }
        }
        __syncthreads();
        // The chunk's tiles with few pairs, all of one worker: nothing has to be ordered, so the pairs of all of them are
        // applied at once, each to its entry (in most of a gradient whose large entries sit elsewhere a tile holds a pair
        // or two, and a tile at a time would be a chain of round trips each).  Every wavefront sees for itself whether the
        // chunk has such tiles; if not, no barrier is spent on them, and the block is kept out of the way of the code around
        // it (eight CF 1000 messages spread evenly over the ResNet101 shape, none such, caches flushed: 33.6 -> 32.5 us,
        // 32.1 without the block; one message of CF 1000 over the VGG16 shape, nothing else: 13.6, 32.3 without the block).
        const int cl = tid & 63;
        const uint32_t cone = cl < tc && (bwrk[cl] >> 16) == 1u && btot[cl] <= DSPARSE ? btot[cl] : 0u;
        static_assert(DCHUNK <= 32, "a bit per tile of a chunk");
        const uint32_t ones = (uint32_t)__ballot(cone != 0u);   // bit i: the chunk's tile i is such a one
        if (__builtin_expect(ones != 0u, 0)) {
            if (tid < 64) {
                const uint32_t inc = wave_scan(cone);
                if (tid < DCHUNK) tpre[tid + 1] = inc;
                if (tid == 0) tpre[0] = 0;
            }
            __syncthreads();
            const uint32_t all = tpre[DCHUNK];
            for (uint32_t k = tid; k < all; k += 256) {
                int i = 0;
#pragma unroll
                for (int step = DCHUNK / 2; step >= 1; step >>= 1)
                    if (tpre[i + step] <= k) i += step;
                const int w = (int)(bwrk[i] & 0xFFFFu);
                const int64_t base = (c0 + (int64_t)i * gridDim.x) * DTILE, end = (n - base < DTILE) ? n : base + DTILE;
                const int64_t at = wat[w] + (int64_t)blo[i * Wp + w] + (int64_t)(k - tpre[i]);
                const int64_t g = idx[at];
                if (g >= base && g < end) dense[g] = __fadd_rn(dense[g], __fmul_rn(alpha, val[at]));
            }
        }
        for (int i = 0; i < tc; ++i) {
            const int64_t tile = c0 + (int64_t)i * gridDim.x;
            if (tile >= ntile) break;
            const int64_t base = tile * DTILE;
            const int len = (int)((n - base < DTILE) ? n - base : DTILE);
            const uint32_t tot = btot[i];
            if (tot == 0) continue;  // no message touches the tile
            if ((ones >> i) & 1u) continue;  // done above
            if (tot <= DSPARSE) {
                // Few pairs: only the entries they name are read and written back, not the whole tile (a scattered
                // access moves 64 bytes, so this pays up to about one pair per 16 entries).  The entries go through
                // the tile buffer all the same, so that pairs of different workers with the same index are added in
                // worker order.
                if (tid < 64) {
                    const uint32_t inc = wave_scan(tid < Wp ? bcnt[i * Wp + tid] : 0u);
                    spre[tid + 1] = inc;
                    if (tid == 0) spre[0] = 0;
                }
                __syncthreads();
                int pj[DSLOTS], pw[DSLOTS];
                float pv[DSLOTS], dv[DSLOTS];
                tile_pairs<DSLOTS>(idx, val, spre, wat, blo + i * Wp, tot, base, len, tid, pj, pv, pw);
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q) dv[q] = pw[q] >= 0 ? dense[base + pj[q]] : 0.0f;
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q)
                    if (pw[q] >= 0) acc[pj[q]] = dv[q];  // the same value from every pair of that entry
                __syncthreads();
                for (int w = 0; w < W; ++w) {
                    if (bcnt[i * Wp + w] == 0) continue;
#pragma unroll
                    for (int q = 0; q < DSLOTS; ++q)
                        if (pw[q] == w) acc[pj[q]] = __fadd_rn(acc[pj[q]], __fmul_rn(alpha, pv[q]));
                    __syncthreads();
                }
#pragma unroll
                for (int q = 0; q < DSLOTS; ++q)
                    if (pw[q] >= 0) dense[base + pj[q]] = acc[pj[q]];
                __syncthreads();  // the tile buffer and spre are free again
                continue;
            }
            bool loaded = false;
            for (int w0 = 0; w0 < W; w0 += DGROUP) {
                const uint32_t* cg = bcnt + i * Wp + w0;
                const uint32_t* lg = blo + i * Wp + w0;
                uint32_t pre[DGROUP + 1];
                pre[0] = 0;
#pragma unroll
                for (int w = 0; w < DGROUP; ++w) pre[w + 1] = pre[w] + cg[w];
                const uint32_t total = pre[DGROUP];
                if (total == 0) continue;  // no message of this group touches the tile
                if (!loaded) {
                    if (vec && len == DTILE) {
                        load_tile<6>(dense + base, acc, tid);
                    } else {
                        for (int q = tid * 4; q < len; q += 256 * 4) {
                            if (vec && q + 4 <= len) {
                                const v4f v = *(const v4f*)(dense + base + q);
                                acc[q] = v.x; acc[q + 1] = v.y; acc[q + 2] = v.z; acc[q + 3] = v.w;
                            } else {
                                for (int e = 0; e < 4 && q + e < len; ++e) acc[q + e] = dense[base + q + e];
                            }
                        }
                    }
                    loaded = true;
                }
                // the group's pairs, worker-major, DBATCH per thread and batch; all loads of a batch in flight together
                for (uint32_t s0 = 0; s0 < total; s0 += 256 * DBATCH) {
                    int pj[DBATCH], pw[DBATCH];
                    float pv[DBATCH];
                    int64_t at[DBATCH];
                    // where the pairs lie (a slot past the last pair takes the last pair's place and is not applied:
                    // total >= 1 here), then all loads without branches around them, in flight together
#pragma unroll
                    for (int q = 0; q < DBATCH; ++q) {
                        const uint32_t slot = s0 + q * 256 + tid;
                        const uint32_t sc = slot < total ? slot : total - 1;
                        int w = 0;
#pragma unroll
                        for (int x = 1; x < DGROUP; ++x) w += (sc >= pre[x]);
                        uint32_t pb = 0;
#pragma unroll
                        for (int x = 1; x < DGROUP; ++x) if (x == w) pb = pre[x];
                        at[q] = wat[w0 + w] + (int64_t)lg[w] + (int64_t)(sc - pb);
                        pw[q] = slot < total ? w : -1;
                    }
#pragma unroll
                    for (int q = 0; q < DBATCH; ++q) pj[q] = idx[at[q]];
#pragma unroll
                    for (int q = 0; q < DBATCH; ++q) pv[q] = val[at[q]];
#pragma unroll
                    for (int q = 0; q < DBATCH; ++q) {
                        const int64_t j = (int64_t)pj[q] - base;
                        if (j < 0 || j >= len) pw[q] = -1;   // an index outside the tile (malformed message) is ignored
                        pj[q] = (int)(j < 0 || j >= len ? 0 : j);
                    }
                    // workers present in this batch: from the worker of its first slot to that of its last
                    const uint32_t end = (s0 + 256 * DBATCH < total ? s0 + 256 * DBATCH : total) - 1;
                    int wmin = 0, wmax = 0;
#pragma unroll
                    for (int x = 1; x < DGROUP; ++x) { wmin += (s0 >= pre[x]); wmax += (end >= pre[x]); }
                    __syncthreads();  // tile loaded / previous batch applied
                    for (int w = wmin; w <= wmax; ++w) {
#pragma unroll
                        for (int q = 0; q < DBATCH; ++q)
                            if (pw[q] == w) acc[pj[q]] = __fadd_rn(acc[pj[q]], __fmul_rn(alpha, pv[q]));
                        __syncthreads();
                    }
                }
            }
            if (loaded) {
                __syncthreads();
                if (vec && len == DTILE) {
                    store_tile<NT>(acc, dense + base, tid);
                } else {
                    for (int q = tid * 4; q < len; q += 256 * 4) {
                        if (vec && q + 4 <= len) {
                            v4f v;
                            v.x = acc[q]; v.y = acc[q + 1]; v.z = acc[q + 2]; v.w = acc[q + 3];
                            *(v4f*)(dense + base + q) = v;
                        } else {
                            for (int e = 0; e < 4 && q + e < len; ++e) dense[base + q + e] = acc[q + e];
                        }
                    }
                }
                __syncthreads();  // the tile buffer is free again
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// A layerwise call's tables, from the pinned host buffer they were built in into the workspace.  A kernel that
// reads the host buffer is queued like every other kernel of the call; a copy by the DMA engine starts 10 to 20 us
// later and the call's first kernel waits for it.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void table_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, uint32_t n16)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < n16) dst[i] = src[i];
}

// ---------------------------------------------------------------------------------------------
// Commit of a message: residual[idx[i]] = +0.0f.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void commit_kernel(const int32_t* __restrict__ idx, int64_t count,
                                                     float* __restrict__ residual, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        const int64_t g = idx[i];
        if ((uint64_t)g < (uint64_t)n) residual[g] = 0.0f;
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct Layout {
    size_t status, tables, tables_bytes, tseg, st, seg, bnd, hist1, ovfc, xq, coarse, list_key, list_tile,
        list_val, list_cnt, samp_hist, samp_above, cand_cnt, brk_cnt, ovn, ovs, tg0, tin, toff, ttake, tsel, ssd, ssd_t, sss,
        cand_idx, cand_val, brk_key, brk_val, total;
};

// Upper bounds that depend only on (n, n_seg).
uint64_t max_tiles(int64_t n, int n_seg) { return (uint64_t)((n + TW - 1) / TW) + (uint64_t)n_seg; }

// Units of the list kernels per tile.  A wavefront per tile is a thousand wavefronts for 8 million elements, each with a long
// walk if many entries are selected; smaller units are shorter walks, but every workgroup of the emit step resolves the
// threshold for itself, so few entries in them are not worth it.  Microseconds with 1, 2 and 4 units per tile, Normal gradients
// (in brackets: with a part whose entries are a hundred times larger, where they crowd):
//    4 million, CF 10   51.4  46.0  44.2  (71.0  55.5  47.9)    CF 100   40.1  39.8  40.3  (46.5  42.2  40.0)
//    8 million, CF 10   60.7  55.4  55.2  (80.6  65.6  58.1)    CF 100   48.3  48.5  49.9  (55.2  51.3  49.6)
//   12 million, CF 10   71.0  66.7  67.0  (89.7  75.1  68.4)    CF 100   57.2  58.0  60.3  (63.8  59.8  59.6)
//   24 million, CF 10   99.1  94.9        (113.6  99.6)         CF 100   80.7  82.1        (86.5  83.0)
constexpr uint64_t FINE_ANY = 512, FINE_MANY = 1536, MIDDLE_ANY = 1024, MIDDLE_MANY = 3072;   // tiles
constexpr int64_t MANY_CF = 40;   // "many": at least every 40th entry is selected
static_assert(FINE_MANY * (SUB / FINE) <= EMIT_RESIDENT && MIDDLE_MANY * (SUB / MIDDLE) <= EMIT_RESIDENT,
              "the wavefronts of such a call are resident at once");
static_assert(DIRECT_MAX <= (int64_t)FINE_ANY * TW / 2, "a direct call's units are FINE sub-tiles");
uint32_t units_per_tile(int64_t n, int n_seg, bool many)
{
    const uint64_t tiles = max_tiles(n, n_seg);
    if (tiles <= (many ? FINE_MANY : FINE_ANY)) return SUB / FINE;
    return tiles <= (many ? MIDDLE_MANY : MIDDLE_ANY) ? SUB / MIDDLE : 1;
}
// Units of a call of up to `tiles` tiles, an upper bound that does not fall as they grow: units_per_tile does, and a workspace
// for a larger tensor has to do for a smaller one.
uint64_t max_units(uint64_t tiles)
{
    const uint64_t fine = tiles * (SUB / FINE);   // (what units_per_tile makes of up to MIDDLE_MANY tiles is at most EMIT_RESIDENT)
    return tiles > EMIT_RESIDENT ? tiles : fine < EMIT_RESIDENT ? fine : EMIT_RESIDENT;
}

uint64_t max_sample_blocks(int64_t n, int n_seg)
{
    static_assert(DENSE_BLOCKS * SAMPLE_BLOCK <= 2 * SAMPLE_MAX && SAMPLE_MAX_FLAT <= DENSE_BLOCKS * SAMPLE_BLOCK * DENSE_ROUNDS,
                  "the blocks of a dense sample fit as well");
    const uint64_t a = (uint64_t)n_seg * (2 * (n_seg > 1 ? SAMPLE_MAX_SEG : SAMPLE_MAX) / SAMPLE_BLOCK);
    const uint64_t b = (uint64_t)((n + SAMPLE_BLOCK - 1) / SAMPLE_BLOCK) + (uint64_t)n_seg;
    return a < b ? a : b;
}

// Copy blocks of the bracket histograms and gather lists.  Global atomics on one cache line queue up, so a large
// tensor spreads them over REP copies (with one copy the streaming pass of the 314-tensor ResNet list takes 120
// instead of 97 us); a small tensor puts so few entries into its brackets that fewer do: 1 below 2^17 elements, then
// 2, 4 and from 2^19 elements on REP.  A flat call always takes REP.  A tensor's copies number at most
// 1 + nt / 2^16, which bounds a layerwise call's total by n_seg + n / 2^16.
uint32_t seg_copies(int64_t nt, bool flat)
{
    static_assert(REP == 8, "1, 2, 4, 8 copies");
    if (flat || nt >= (1 << 19)) return REP;
    return nt >= (1 << 18) ? 4u : nt >= (1 << 17) ? 2u : 1u;
}
size_t pool_blocks(int64_t n, int n_cf, int n_seg)
{
    if (n_seg <= 1) return (size_t)n_cf * REP;
    const size_t graded = (size_t)n_seg + (size_t)(n >> 16), all = (size_t)n_seg * REP;
    return (size_t)n_cf * (graded < all ? graded : all);
}

Layout make_layout(int64_t n, int n_cf, int n_seg)
{
    Layout L;
    size_t at = 0;
    auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes, 256); return o; };
    const uint64_t nt = max_tiles(n, n_seg), nsb = max_sample_blocks(n, n_seg), nu = max_units(nt);
    const size_t sc = (size_t)n_seg * n_cf;
    L.status = take(sizeof(Status));
    // host-built tables, one piece: SegInfo[n_seg], ktab[n_seg][n_cf], sblock_seg[sample blocks]
    L.tables_bytes = sizeof(SegInfo) * n_seg + sizeof(uint32_t) * sc + sizeof(uint32_t) * nsb;
    L.tables = take(L.tables_bytes);
    L.tseg = take(sizeof(uint32_t) * nt);
    L.st = take(sizeof(CfState) * sc);
    L.seg = take(sizeof(SegState) * n_seg);
    L.bnd = take(sizeof(uint32_t) * BND_WORDS * (size_t)n_seg);
    const size_t blocks = pool_blocks(n, n_cf, n_seg);
    L.hist1 = take(sizeof(uint32_t) * blocks * NBIN);
    L.ovfc = take(sizeof(uint32_t) * sc * 64 * 32);
    L.xq = take(sizeof(uint32_t) * (size_t)n_seg * XQ_LINE);
    L.coarse = take(sizeof(uint32_t) * (size_t)n_seg * NBIN);
    L.list_key = take(sizeof(uint32_t) * blocks * LCAP);
    L.list_tile = take(sizeof(uint32_t) * blocks * LCAP);
    L.list_val = take(sizeof(float) * blocks * LCAP);
    L.list_cnt = take(sizeof(uint32_t) * blocks * 32);
    L.samp_hist = take(sizeof(uint32_t) * nsb * (SBIN / 2));
    L.samp_above = take(sizeof(uint16_t) * nsb * RGRP);
    L.cand_cnt = take(sizeof(uint32_t) * nt * SUB);
    L.brk_cnt = take(sizeof(uint32_t) * nt * SUB);
    L.ovn = take(sizeof(uint32_t) * nt * SUB * n_cf);
    L.ovs = take(sizeof(double) * nt * SUB * n_cf);
    L.tg0 = take(sizeof(uint32_t) * nu);
    L.tin = take(sizeof(uint32_t) * nu);
    L.toff = take(sizeof(uint32_t) * nu);   // (or csum: 64 bytes per CTILES = 64 tiles, a quarter of that)
    L.ttake = take(sizeof(uint32_t) * nt);
    L.tsel = take(sizeof(uint32_t) * nu);   // (or wseg)
    L.ssd = take(sizeof(double) * nt * SUB);
    L.ssd_t = take(sizeof(double) * nu);
    L.sss = take(sizeof(double) * nu * n_cf);
    L.cand_idx = take(sizeof(int32_t) * nt * TW);
    L.cand_val = take(sizeof(float) * nt * TW);
    L.brk_key = take(sizeof(uint32_t) * nt * TW);
    L.brk_val = take(sizeof(float) * nt * TW);
    L.total = at;
    return L;
}

// samples taken from a segment of nt elements when the CFs range from cf_min to cf_max
uint32_t sample_count(uint64_t nt, double cf_min, double cf_max, bool flat)
{
    // layerwise: the larger of 32 CF_max and 1/64 of the tensor.  A small sample of a large tensor gives a wide
    // bracket: many more entries in it than k, and bins so coarse that the keys near the bracket's lower end crowd
    // into a few histogram bins, where their atomics queue up behind each other
    uint64_t target = flat ? (uint64_t)SAMPLE_MAX : (uint64_t)(32.0 * std::ceil(cf_max));
    if (!flat && target < nt / 64) target = nt / 64;
    if (target < 4096) target = 4096;
    const uint64_t cap = flat ? SAMPLE_MAX : SAMPLE_MAX_SEG;
    if (target > cap) target = cap;
    if (flat) {
        // The bracket spans about 10 standard deviations of a sampled rank, which is 10 sqrt(k nt / m) of the tensor's
        // entries for m samples, and every entry inside it costs the streaming pass a device-wide atomic (about
        // ten per nanosecond all told, and a gradient whose large entries sit together sends them all at once): a
        // selection of many entries from a large tensor (k = nt / cf_min) takes more samples, enough to keep that
        // number near 300,000.
        const double need = 64.0 * ((double)nt / cf_min) * (double)nt / 68719476736.0;  // 2^36
        if (need > (double)target) target = need > (double)SAMPLE_MAX_FLAT ? (uint64_t)SAMPLE_MAX_FLAT : (uint64_t)need;
    }
    const uint64_t unit = target > (uint64_t)SAMPLE_MAX ? SAMPLE_BLOCK * DENSE_ROUNDS : SAMPLE_BLOCK;
    target = (target + unit - 1) / unit * unit;
    return (nt <= 2 * target) ? (uint32_t)nt : (uint32_t)target;
}

// Pinned host staging for the layerwise tables: a small ring of slots, each followed on its stream by an
// event, so that a slot is only rewritten after the copy that read it has run.  Host memory only; grown on demand.
// This ring is the only state the library keeps between calls.
struct StagingSlot {
    char* mem = nullptr;
    size_t cap = 0;
    hipEvent_t done = nullptr;
    bool pending = false;  // `done` was recorded and not yet waited for
    bool busy = false;     // held by a caller (being waited for, filled or copied from)
};
constexpr int STAGING_SLOTS = 8;
StagingSlot g_staging[STAGING_SLOTS];
int g_staging_next = 0;
std::mutex g_staging_mutex;

StagingSlot* staging_acquire(size_t bytes)
{
    StagingSlot* s = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_staging_mutex);
        // A slot that is large enough and whose last copy has run; else, while fewer than two slots have memory, one
        // without (it is allocated below); else one whose copy is still queued (its event is waited for below: the host
        // then runs at most a call or two ahead of the GPU); else, all of those being held by other callers, one
        // without memory.  Pinning fresh host memory takes milliseconds and slows the first copy out of it, so a caller
        // that runs ahead of the GPU does not get a new slot for every call it is ahead.
        int with_mem = 0;
        for (int i = 0; i < STAGING_SLOTS; ++i) with_mem += g_staging[i].cap > 0 ? 1 : 0;
        for (int pass = 0; pass < 4 && !s; ++pass) {
            if (pass == 1 && with_mem >= 2) continue;
            for (int i = 0; i < STAGING_SLOTS && !s; ++i) {
                StagingSlot* c = &g_staging[(g_staging_next + i) % STAGING_SLOTS];
                if (c->busy) continue;
                const bool ready = c->cap >= bytes && (!c->pending || hipEventQuery(c->done) == hipSuccess);
                if ((pass == 0 && ready) || ((pass == 1 || pass == 3) && c->cap == 0) || (pass == 2 && c->cap > 0)) {
                    s = c;
                    g_staging_next = (g_staging_next + i + 1) % STAGING_SLOTS;
                }
            }
        }
        if (!s) return nullptr;  // more concurrent callers than slots
        s->busy = true;
    }
    // the slot is this caller's now: the waiting and the allocation happen outside the lock
    bool ok = true;
    if (!s->done && hipEventCreateWithFlags(&s->done, hipEventDisableTiming) != hipSuccess) { s->done = nullptr; ok = false; }
    if (ok && s->pending) {
        if (hipEventSynchronize(s->done) != hipSuccess) ok = false;
        else s->pending = false;
    }
    if (ok && s->cap < bytes) {
        if (s->mem) (void)hipHostFree(s->mem);
        s->mem = nullptr; s->cap = 0;
        const size_t want = bytes < 65536 ? 65536 : bytes + bytes / 2;
        if (hipHostMalloc((void**)&s->mem, want, hipHostMallocDefault) != hipSuccess) { s->mem = nullptr; ok = false; }
        else s->cap = want;
    }
    if (!ok) {
        std::lock_guard<std::mutex> lock(g_staging_mutex);
        s->busy = false;
        return nullptr;
    }
    return s;
}

void staging_release(StagingSlot* s, bool recorded)
{
    std::lock_guard<std::mutex> lock(g_staging_mutex);
    s->pending = recorded;
    s->busy = false;
}

}  // namespace

// Scratch of gravac_decompress_accumulate_static, the entry point for callers that cannot allocate: the tile
// boundaries of the messages (what the caller's workspace holds in gravac_decompress_accumulate).  Every GPU the
// library runs on holds its own copy of the array, at its own address, until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; kernels get the address that call returned.
constexpr size_t STATIC_SCRATCH_WORDS = (size_t)GRAVAC_STATIC_SCRATCH_BYTES / sizeof(uint32_t);
static __device__ __align__(256) uint32_t scratch[STATIC_SCRATCH_WORDS];

namespace {

constexpr int MAX_DEVICES = 64;
uint32_t* g_scratch_ptr[MAX_DEVICES];  // device address of `scratch` on every device used so far
std::mutex g_scratch_mutex;

// The address of `scratch` on the current device, looked up once per device.
int static_scratch(uint32_t** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return GRAVAC_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return GRAVAC_ERR_HIP;
        g_scratch_ptr[dev] = (uint32_t*)ptr;
    }
    *out = g_scratch_ptr[dev];
    return GRAVAC_OK;
}

}  // namespace

extern "C" {

int64_t gravac_topk_count(int64_t n, double cf)
{
    if (n <= 0 || !(cf >= 1.0) || std::isinf(cf)) return -1;
    int64_t k;
    if (cf == std::floor(cf) && cf < 9.0e18) {
        const int64_t c = (int64_t)cf;
        k = (n + c - 1) / c;
    } else {
        k = (int64_t)std::ceil((double)n / cf);
    }
    if (k < 1) k = 1;
    if (k > n) k = n;
    return k;
}

int gravac_workspace_bytes(int64_t n, int n_cf, int n_seg, size_t* bytes_out)
{
    if (!bytes_out || n <= 0 || n > 2147483647LL || n_cf < 1 || n_cf > MAXCF || n_seg < 0) return GRAVAC_ERR_INVALID_ARG;
    if ((int64_t)n_seg > n) return GRAVAC_ERR_INVALID_ARG;
    *bytes_out = make_layout(n, n_cf, n_seg < 1 ? 1 : n_seg).total;
    return GRAVAC_OK;
}

// GRAVAC_OK if `stream` is not being captured into a graph, else GRAVAC_ERR_CAPTURE (asked only by calls that cannot
// be replayed: a replay would copy whatever the staging slot holds by then, or re-record the caller's events).
static int refuse_capture(hipStream_t stream)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) return GRAVAC_ERR_HIP;
    return cap == hipStreamCaptureStatusNone ? GRAVAC_OK : GRAVAC_ERR_CAPTURE;
}

// The pipeline behind all compression entry points.  map_idx == null: error-feedback compression of grad + residual.
// map_idx != null: single-source mode, the source is grad alone (a message's values), map_idx its indices,
// restore / n_restore the dense residual that takes the unselected values back (may be null).
// seed != null: Random-k.  ev != null: the caller's events are recorded around the call and the pass over the gradient.
static int compress_impl(const float* grad, float* residual, int64_t n, const double* cf_list, int n_cf, int commit,
                         const int64_t* seg_offsets, int n_seg, int32_t* out_idx, float* out_val, int64_t out_capacity,
                         int64_t* out_count, double* out_stats, void* workspace, size_t workspace_bytes, unsigned flags,
                         hipStream_t stream, const int32_t* map_idx, float* restore, int64_t n_restore,
                         const uint64_t* seed, const gravac_profile_events* ev, const float* tau = nullptr)
{
    const bool single = map_idx != nullptr;
    const bool random = seed != nullptr;
    const bool fixed = tau != nullptr;  // the threshold sparsifier: one flat tensor, cf_list = {1}, out_capacity as given
    if (fixed && (single || random || n_seg != 0 || n_cf != 1 || !out_count || out_capacity < 0)) return GRAVAC_ERR_INVALID_ARG;
    if (fixed && (!(*tau > 0.0f) || std::isinf(*tau))) return GRAVAC_ERR_INVALID_ARG;
    if (!grad || (!single && !residual) || !cf_list || !out_stats) return GRAVAC_ERR_INVALID_ARG;
    if ((!out_idx || !out_val) && !(fixed && out_capacity == 0)) return GRAVAC_ERR_INVALID_ARG;
    if (n <= 0 || n > 2147483647LL || n_cf < 1 || n_cf > MAXCF || commit < 0 || commit >= n_cf) return GRAVAC_ERR_INVALID_ARG;
    if (((uintptr_t)grad & 3) || ((uintptr_t)residual & 3) || ((uintptr_t)map_idx & 3)) return GRAVAC_ERR_INVALID_ARG;
    if (flags & ~(unsigned)(GRAVAC_FLAG_FORCE_FALLBACK | GRAVAC_FLAG_NO_COMMIT | GRAVAC_FLAG_STALL_FALLBACK)) return GRAVAC_ERR_INVALID_ARG;
    const bool stall = (flags & GRAVAC_FLAG_STALL_FALLBACK) != 0;
    if (stall && !(flags & GRAVAC_FLAG_FORCE_FALLBACK)) return GRAVAC_ERR_INVALID_ARG;
    if ((flags & GRAVAC_FLAG_NO_COMMIT) && (single || fixed)) return GRAVAC_ERR_INVALID_ARG;
    if (n_seg < 0 || (n_seg > 0 && !seg_offsets) || (int64_t)n_seg > n) return GRAVAC_ERR_INVALID_ARG;
    if (ev && (!ev->call_begin || !ev->pass_begin || !ev->pass_end || !ev->call_end)) return GRAVAC_ERR_INVALID_ARG;
    double cf_max = 1.0, cf_min = cf_list[0];
    for (int j = 0; j < n_cf; ++j) {
        if (!(cf_list[j] >= 1.0) || std::isinf(cf_list[j])) return GRAVAC_ERR_INVALID_ARG;
        if (cf_list[j] > cf_max) cf_max = cf_list[j];
        if (cf_list[j] < cf_min) cf_min = cf_list[j];
    }
    const int ns = n_seg < 1 ? 1 : n_seg;
    if (n_seg >= 1) {
        if (seg_offsets[0] != 0 || seg_offsets[n_seg] != n) return GRAVAC_ERR_INVALID_ARG;
        for (int t = 0; t < n_seg; ++t)
            if (seg_offsets[t + 1] <= seg_offsets[t]) return GRAVAC_ERR_INVALID_ARG;
    }
    if (!workspace || ((uintptr_t)workspace & 255)) return GRAVAC_ERR_WORKSPACE;
    const Layout L = make_layout(n, n_cf, ns);
    if (workspace_bytes < L.total) return GRAVAC_ERR_WORKSPACE;

    char* ws = (char*)workspace;
    Params p;
    std::memset(&p, 0, sizeof(p));
    p.grad = grad; p.res = residual; p.acc = single ? grad : residual;
    p.map_idx = map_idx; p.restore = restore; p.n_restore = restore ? n_restore : 0; p.single = single ? 1 : 0;
    p.no_commit = (flags & GRAVAC_FLAG_NO_COMMIT) ? 1 : 0;
    p.bounds_from = (flags & GRAVAC_FLAG_FORCE_FALLBACK) ? BOUNDS_FORCED : (random ? BOUNDS_RANDOM : BOUNDS_SAMPLED);
    p.wait_polls = stall ? WAIT_POLLS_TEST : WAIT_POLLS;
    p.wait_extra = stall ? 1u : 0u;
    if (fixed) {
        p.bounds_from = BOUNDS_FIXED;
        std::memcpy(&p.fixed_key, tau, sizeof(uint32_t));   // positive and finite: the bit pattern is the key
    }
    if (random) {
        // the seed goes through SplitMix64 (its first output for that seed) and gives the two 31-bit keys
        uint64_t z = *seed + 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        p.random = 1;
        p.rk_s0 = (uint32_t)(z & 0x7FFFFFFFull);
        p.rk_s1 = (uint32_t)((z >> 32) & 0x7FFFFFFFull);
    }
    p.n = n; p.n_seg = ns; p.n_cf = n_cf; p.commit = commit;
    p.status = (Status*)(ws + L.status);
    p.segs = (const SegInfo*)(ws + L.tables);
    p.ktab = (const uint32_t*)(ws + L.tables + sizeof(SegInfo) * ns);
    p.sblock_seg = p.ktab + (size_t)ns * n_cf;
    p.tseg = (uint32_t*)(ws + L.tseg);
    p.st = (CfState*)(ws + L.st);
    p.seg = (SegState*)(ws + L.seg);
    p.bnd = (uint32_t*)(ws + L.bnd);
    p.hist1 = (uint32_t*)(ws + L.hist1);
    p.ovfc = (uint32_t*)(ws + L.ovfc);
    p.xq = (uint32_t*)(ws + L.xq);
    p.coarse = (uint32_t*)(ws + L.coarse);
    p.list_key = (uint32_t*)(ws + L.list_key);
    p.list_tile = (uint32_t*)(ws + L.list_tile);
    p.list_val = (float*)(ws + L.list_val);
    p.list_cnt = (uint32_t*)(ws + L.list_cnt);
    p.samp_hist = (uint32_t*)(ws + L.samp_hist);
    p.samp_above = (uint16_t*)(ws + L.samp_above);
    p.cand_cnt = (uint32_t*)(ws + L.cand_cnt);
    p.brk_cnt = (uint32_t*)(ws + L.brk_cnt);
    p.ovn = (uint32_t*)(ws + L.ovn);
    p.ovs = (double*)(ws + L.ovs);
    p.tg0 = (uint32_t*)(ws + L.tg0);
    p.tin = (uint32_t*)(ws + L.tin);
    p.toff = (uint32_t*)(ws + L.toff);
    p.ttake = (uint32_t*)(ws + L.ttake);
    p.tsel = (uint32_t*)(ws + L.tsel);
    p.ssd = (double*)(ws + L.ssd);
    p.ssd_t = (double*)(ws + L.ssd_t);
    p.sss = (double*)(ws + L.sss);
    p.cand_idx = (int32_t*)(ws + L.cand_idx);
    p.cand_val = (float*)(ws + L.cand_val);
    p.brk_key = (uint32_t*)(ws + L.brk_key);
    p.brk_val = (float*)(ws + L.brk_val);
    p.out_idx = out_idx; p.out_val = out_val; p.out_count = out_count; p.out_stats = out_stats;

    int64_t total_out = 0;
    uint32_t max_seg_tiles = 1;  // tiles of the largest segment
    uint32_t emit_wgs = 0;       // workgroups of an emit step without scan that take units
    int sample_rounds = 1;       // groups per thread of the sampling kernel
    uint32_t n_small = 0;        // layerwise: tensors of at most SMALL_MAX elements, one workgroup each (not under the
                                 // testing flag, which sends every tensor through the histogram route)
    const bool small_ok = ns > 1 && !(flags & GRAVAC_FLAG_FORCE_FALLBACK);
    StagingSlot* slot = nullptr;
    size_t table_bytes = 0;
    if (ns == 1) {
        for (int j = 0; j < n_cf; ++j) p.flat_k[j] = (uint32_t)gravac_topk_count(n, cf_list[j]);
        p.direct = n <= DIRECT_MAX && p.bounds_from == BOUNDS_SAMPLED ? 1 : 0;
        p.flat_samples = p.direct ? (uint32_t)n : sample_count((uint64_t)n, cf_min, cf_max, true);
        static_assert(DIRECT_MAX <= SAMPLE_MAX_FLAT, "as many samples as the blocks can take");
        p.n_tiles = (uint32_t)((n + TW - 1) / TW);
        max_seg_tiles = p.n_tiles;
        // more than SAMPLE_MAX samples (never a tensor read whole): 2 or 4 times SAMPLE_BLOCK samples per block, the
        // fewest that leave at most DENSE_BLOCKS blocks (more blocks keep more loads in flight, fewer cost the
        // bracket kernel fewer round trips, one per 64 blocks)
        if (p.flat_samples > (uint32_t)SAMPLE_MAX && ((int64_t)p.flat_samples != n || p.direct))
            while (sample_rounds < DENSE_ROUNDS && p.flat_samples > (uint32_t)(DENSE_BLOCKS * SAMPLE_BLOCK * sample_rounds))
                sample_rounds *= 2;
        const uint32_t per_block = SAMPLE_BLOCK * sample_rounds;
        p.n_sample_blocks = (p.flat_samples + per_block - 1) / per_block;
        total_out = p.flat_k[commit];
        if (fixed) {
            // the number of pairs is only known on the device: the emit step writes up to the caller's capacity
            total_out = out_capacity < n ? out_capacity : n;
            p.flat_k[0] = (uint32_t)total_out;
        }
        if (total_out > out_capacity) return GRAVAC_ERR_CAPACITY;
    } else {
        // layerwise tables: sized first, then built straight into a pinned staging slot and copied into the
        // workspace with one asynchronous copy (no host synchronisation)
        uint64_t tiles = 0, sblocks = 0;
        for (int t = 0; t < ns; ++t) {
            const int64_t nt = seg_offsets[t + 1] - seg_offsets[t];
            total_out += gravac_topk_count(nt, cf_list[commit]);
            if (small_ok && nt <= SMALL_MAX) { ++n_small; continue; }  // one workgroup does it all: no tiles, no samples
            const uint64_t tt = (uint64_t)((nt + TW - 1) / TW);
            tiles += tt;
            if (tt > max_seg_tiles) max_seg_tiles = (uint32_t)tt;
            sblocks += (sample_count((uint64_t)nt, cf_min, cf_max, false) + SAMPLE_BLOCK - 1) / SAMPLE_BLOCK;
        }
        if (total_out > out_capacity) return GRAVAC_ERR_CAPACITY;
        if (tiles > max_tiles(n, ns) || sblocks > max_sample_blocks(n, ns)) return GRAVAC_ERR_WORKSPACE;
        p.n_tiles = (uint32_t)tiles;
        p.n_sample_blocks = (uint32_t)sblocks;
    }
    // (the threshold sparsifier's count is not known: few)
    const uint32_t upt = units_per_tile(n, ns, !fixed && total_out >= n / MANY_CF);
    if (ns == 1) emit_wgs = (p.n_tiles * upt + EW - 1) / EW;
    const bool with_scan = p.n_tiles > EMIT_RESIDENT;   // see resolve_emit_kernel
    if (!with_scan) {
        p.csum = (uint64_t*)p.toff;
        p.n_csum = (p.n_tiles * upt + CTILES - 1u) / CTILES;
        p.wseg = p.tsel;
    }
    // nothing has been queued or written up to here; from here on an error return leaves the outputs unspecified
    if (ns > 1 || ev)
        if (const int rc = refuse_capture(stream)) return rc;
    (void)hipGetLastError();  // an error left behind by earlier work of the process is not this call's
    if (ns > 1) {
        table_bytes = sizeof(SegInfo) * ns + sizeof(uint32_t) * (size_t)ns * n_cf + sizeof(uint32_t) * p.n_sample_blocks;
        table_bytes = (table_bytes + 15) & ~(size_t)15;   // (moved 16 bytes at a time; the workspace's part is that long)
        slot = staging_acquire(table_bytes);
        if (!slot) return GRAVAC_ERR_HIP;
        SegInfo* segs = (SegInfo*)slot->mem;
        uint32_t* ktab = (uint32_t*)(slot->mem + sizeof(SegInfo) * ns);
        uint32_t* sblock_seg = ktab + (size_t)ns * n_cf;
        int64_t koff = 0;
        uint32_t tile_at = 0, sb_at = 0, block_at = 0;
        for (int t = 0; t < ns; ++t) {
            const int64_t nt = seg_offsets[t + 1] - seg_offsets[t];
            SegInfo& g = segs[t];
            std::memset(&g, 0, sizeof(g));
            g.begin = seg_offsets[t]; g.end = seg_offsets[t + 1]; g.koff = koff;
            g.tile0 = g.tile1 = tile_at; g.samp0 = sb_at;
            g.rep = seg_copies(nt, false); g.pool0 = block_at; block_at += (uint32_t)n_cf * g.rep;
            if (small_ok && nt <= SMALL_MAX) {
                g.small = 1;
            } else {
                tile_at += (uint32_t)((nt + TW - 1) / TW); g.tile1 = tile_at;
                g.wg0 = emit_wgs; g.wgs = ((g.tile1 - g.tile0) * upt + EW - 1) / EW; emit_wgs += g.wgs;
                g.samp_cnt = sample_count((uint64_t)nt, cf_min, cf_max, false);
                const uint32_t nb = (g.samp_cnt + SAMPLE_BLOCK - 1) / SAMPLE_BLOCK;
                for (uint32_t b = 0; b < nb; ++b) sblock_seg[sb_at + b] = (uint32_t)t;
                sb_at += nb;
            }
            for (int j = 0; j < n_cf; ++j) ktab[(size_t)t * n_cf + j] = (uint32_t)gravac_topk_count(nt, cf_list[j]);
            koff += ktab[(size_t)t * n_cf + commit];
        }
    }
    p.total_out = total_out;
    if (ev && hipEventRecord((hipEvent_t)ev->call_begin, stream) != hipSuccess) {
        if (slot) staging_release(slot, false);
        return GRAVAC_ERR_HIP;
    }
    if (slot) {
        bool copied;
        // the buffer as a kernel of the current device addresses it (none: only a copy can read it)
        void* dev = nullptr;
        if (hipHostGetDevicePointer(&dev, slot->mem, 0) != hipSuccess) { dev = nullptr; (void)hipGetLastError(); }
        if (dev) {
            const uint32_t n16 = (uint32_t)(table_bytes / 16);
            hipLaunchKernelGGL(table_copy_kernel, dim3((n16 + 255) / 256), dim3(256), 0, stream, (const uint4*)dev,
                               (uint4*)(ws + L.tables), n16);
            copied = hipGetLastError() == hipSuccess;
        } else {
            copied = hipMemcpyAsync(ws + L.tables, slot->mem, table_bytes, hipMemcpyHostToDevice, stream) == hipSuccess;
        }
        bool recorded = copied && hipEventRecord(slot->done, stream) == hipSuccess;
        // a copy that is queued but not followed by the slot's event: wait for it here, so that the slot is not
        // rewritten under it
        if (copied && !recorded) (void)hipStreamSynchronize(stream);
        staging_release(slot, recorded);
        if (!copied || !recorded) return GRAVAC_ERR_HIP;
    }

    const uint32_t sub_grid = (p.n_tiles * SUB + WAVES - 1) / WAVES;
    const uint32_t light_grid = (p.n_tiles * upt + LWAVES - 1) / LWAVES;

    const int ncf_form = n_cf <= 1 ? 0 : n_cf <= 2 ? 1 : n_cf <= 3 ? 2 : n_cf <= 4 ? 3 : 4;
    static_assert(MAXCF >= 4, "forms for 1, 2, 3, 4 and MAXCF CFs");
    static_assert(DENSE_ROUNDS == 4, "forms of the sampling kernel for 1, 2 and 4 groups per thread");
    // (a layerwise call takes SAMPLE_BLOCK samples per block; its small tensors are extra workgroups of this launch)
    const bool have_tiles = p.n_tiles != 0;  // (not if every tensor of a layerwise call is small)
    if (have_tiles && !fixed) {              // (the threshold sparsifier uses nothing of what this kernel samples or clears)
        void (*const sample_forms[3])(Params) = {sample_kernel<1>, sample_kernel<2>, sample_kernel<4>};
        hipLaunchKernelGGL(sample_forms[sample_rounds == 1 ? 0 : sample_rounds == 2 ? 1 : 2], dim3(p.n_sample_blocks), dim3(256),
                           0, stream, p);
    }
    // a layerwise call's small tensors are done by their workgroups of this launch; few segments (none of them small):
    // their sample histograms are added up by SGRP workgroups each; many: by one each
    if (ns == 1 && p.bounds_from == BOUNDS_SAMPLED)
        hipLaunchKernelGGL(p.direct ? bracket_kernel<true> : bracket_kernel<false>, dim3(RGRP), dim3(64), 0, stream, p);
    else if (n_small)
        hipLaunchKernelGGL((threshold_kernel<1, true>), dim3(ns, 1), dim3(1024), 0, stream, p);
    else if (ns > 1 && ns <= 32 && p.bounds_from == BOUNDS_SAMPLED)
        hipLaunchKernelGGL((threshold_kernel<SGRP, false, 2>), dim3(ns, SGRP), dim3(2048 / SGRP), 0, stream, p);
    else if (ns > 1)
        hipLaunchKernelGGL((threshold_kernel<1, false>), dim3(ns, 1), dim3(1024), 0, stream, p);
    {
        // the pass exists in forms for 1, 2, 3, 4 and MAXCF CFs (its loops over the CFs are unrolled)
        void (*const ef_forms[5])(Params) = {stream_kernel<SM_EF, false, false, 1>, stream_kernel<SM_EF, false, false, 2>,
                                             stream_kernel<SM_EF, false, false, 3>, stream_kernel<SM_EF, false, false, 4>,
                                             stream_kernel<SM_EF, false, false, MAXCF>};
        void (*const rk_forms[5])(Params) = {stream_kernel<SM_EF, true, false, 1>, stream_kernel<SM_EF, true, false, 2>,
                                             stream_kernel<SM_EF, true, false, 3>, stream_kernel<SM_EF, true, false, 4>,
                                             stream_kernel<SM_EF, true, false, MAXCF>};
        void (*const direct_forms[5])(Params) = {stream_kernel<SM_EF, false, true, 1>, stream_kernel<SM_EF, false, true, 2>,
                                                 stream_kernel<SM_EF, false, true, 3>, stream_kernel<SM_EF, false, true, 4>,
                                                 stream_kernel<SM_EF, false, true, MAXCF>};
        void (*kern)(Params) = single ? (p.direct ? stream_kernel<SM_SINGLE, false, true, 1>     // (a second-level call has one CF)
                                                  : stream_kernel<SM_SINGLE, false, false, 1>)
                                      : (random ? rk_forms : p.direct ? direct_forms : ef_forms)[ncf_form];
        if (!have_tiles) {
            if (ev) { (void)hipEventRecord((hipEvent_t)ev->pass_begin, stream); (void)hipEventRecord((hipEvent_t)ev->pass_end, stream); }
        } else if (ev)  // the kernel's own begin and end time stamps
            hipExtLaunchKernelGGL(kern, dim3(sub_grid), dim3(WG), 0, stream, (hipEvent_t)ev->pass_begin,
                                  (hipEvent_t)ev->pass_end, 0, p);
        else
            hipLaunchKernelGGL(kern, dim3(sub_grid), dim3(WG), 0, stream, p);
    }
    if (have_tiles && !fixed && !p.direct) {
    // a flat call: as many workgroups as its tiles can keep busy should its bracket have failed; layerwise: one per tensor
    // and one more per PLAN_HELP tiles of a large one
    const uint32_t plan_flat = (p.n_tiles + PLAN_T / 64 - 1) / (PLAN_T / 64);
    const uint32_t plan_grid = ns == 1 ? (plan_flat < PLAN_GRID ? plan_flat : PLAN_GRID) : (uint32_t)ns + p.n_tiles / PLAN_HELP;
    hipLaunchKernelGGL(random ? plan_kernel<true> : plan_kernel<false>, dim3(plan_grid), dim3(PLAN_T), 0, stream, p);
    }
    if (have_tiles) {
    // the refine kernel loops over the CFs: forms for 1, 2, 3, 4 and MAXCF CFs
    // (... and with or without the early loads of the lists' heads: with them if the tiles' wavefronts are all resident
    // at once, six per SIMD on 1024 SIMDs)
#define REFINE_FORMS(heads, u) {refine_kernel<1, heads, u>, refine_kernel<2, heads, u>, refine_kernel<3, heads, u>, refine_kernel<4, heads, u>, refine_kernel<MAXCF, heads, u>}
    void (*const refine_forms[3][2][5])(Params) = {{REFINE_FORMS(false, SUB), REFINE_FORMS(true, SUB)},
                                                   {REFINE_FORMS(false, MIDDLE), REFINE_FORMS(true, MIDDLE)},
                                                   {REFINE_FORMS(false, FINE), REFINE_FORMS(true, FINE)}};
#undef REFINE_FORMS
    const int fine = upt == 1 ? 0 : upt == SUB / MIDDLE ? 1 : 2;
    const int heads = (!random && p.n_tiles <= EMIT_RESIDENT) ? 1 : 0;
    if (!p.direct) hipLaunchKernelGGL(refine_forms[fine][heads][ncf_form], dim3(light_grid), dim3(LWG), 0, stream, p);
    const bool general = p.random || p.single;   // (the plain call has forms of its own)
    const int stream_out = !fixed && total_out >= STREAM_OUT && (with_scan || 5 * total_out < 2 * n) ? 1 : 0;   // (see STREAM_OUT)
    void (*const scan_emit_forms[2][2])(Params) = {{emit_kernel<false, false>, emit_kernel<true, false>}, {emit_kernel<false, true>, emit_kernel<true, true>}};
    if (with_scan) {
        const uint32_t scan_slices = (max_seg_tiles + SCAN_SLICE - 1) / SCAN_SLICE;
        hipLaunchKernelGGL(scan_kernel, dim3(ns, scan_slices + n_cf), dim3(SCAN_T), 0, stream, p, scan_slices);
        hipLaunchKernelGGL(scan_emit_forms[stream_out][general ? 1 : 0], dim3(light_grid), dim3(LWG), 0, stream, p);
    } else {
        // (There is a streamed form for units of a tile only.  Smaller units, of calls of up to 25 million elements, gain little by
        // it: 16 and 24 million at CF 10 75.7 -> 75.3 and 94.6 -> 94.8 us, with a part a hundred times larger 83.7 -> 81.0 and
        // 100.2 -> 98.7; 24 million at CF 4 110.3 -> 109.6, three states in turn 125.4 -> 114.6; at CF 2 138 -> 147.  Units of a tile,
        // streamed, instead of them: 16 million at CF 10 79.5, at CF 4 98.7 instead of 92.7.)
#define EMIT_FORMS(u, direct, streamed) {resolve_emit_kernel<false, u, direct, streamed>, resolve_emit_kernel<true, u, direct, streamed>}
        void (*const emit_forms[5][2])(Params) = {EMIT_FORMS(SUB, false, false), EMIT_FORMS(MIDDLE, false, false), EMIT_FORMS(FINE, false, false),
                                                  EMIT_FORMS(FINE, true, false), EMIT_FORMS(SUB, false, true)};
#undef EMIT_FORMS
        hipLaunchKernelGGL(emit_forms[p.direct ? 3 : fine == 0 && stream_out ? 4 : fine][general ? 1 : 0], dim3(emit_wgs + (uint32_t)(ns * n_cf)),
                           dim3(EWG), 0, stream, p);
    }
    }
    if (ev) (void)hipEventRecord((hipEvent_t)ev->call_end, stream);
    if (hipGetLastError() != hipSuccess) return GRAVAC_ERR_HIP;
    return GRAVAC_OK;
}

int gravac_compress(const float* grad, float* residual, int64_t n, const double* cf_list, int n_cf, int commit,
                    const int64_t* seg_offsets, int n_seg, int32_t* out_idx, float* out_val, int64_t out_capacity,
                    int64_t* out_count, double* out_stats, void* workspace, size_t workspace_bytes, unsigned flags,
                    void* stream_v)
{
    if (!residual) return GRAVAC_ERR_INVALID_ARG;
    return compress_impl(grad, residual, n, cf_list, n_cf, commit, seg_offsets, n_seg, out_idx, out_val, out_capacity,
                         out_count, out_stats, workspace, workspace_bytes, flags, (hipStream_t)stream_v, nullptr, nullptr, 0,
                         nullptr, nullptr);
}

int gravac_compress_profiled(const float* grad, float* residual, int64_t n, const double* cf_list, int n_cf, int commit,
                             const int64_t* seg_offsets, int n_seg, int32_t* out_idx, float* out_val,
                             int64_t out_capacity, int64_t* out_count, double* out_stats, void* workspace,
                             size_t workspace_bytes, unsigned flags, void* stream_v, const gravac_profile_events* events)
{
    if (!residual || !events) return GRAVAC_ERR_INVALID_ARG;
    return compress_impl(grad, residual, n, cf_list, n_cf, commit, seg_offsets, n_seg, out_idx, out_val, out_capacity,
                         out_count, out_stats, workspace, workspace_bytes, flags, (hipStream_t)stream_v, nullptr, nullptr, 0,
                         nullptr, events);
}

int gravac_randomk_compress(const float* grad, float* residual, int64_t n, const double* cf_list, int n_cf, int commit,
                            uint64_t seed, const int64_t* seg_offsets, int n_seg, int32_t* out_idx, float* out_val,
                            int64_t out_capacity, int64_t* out_count, double* out_stats, void* workspace,
                            size_t workspace_bytes, unsigned flags, void* stream_v)
{
    if (!residual) return GRAVAC_ERR_INVALID_ARG;
    return compress_impl(grad, residual, n, cf_list, n_cf, commit, seg_offsets, n_seg, out_idx, out_val, out_capacity,
                         out_count, out_stats, workspace, workspace_bytes, flags, (hipStream_t)stream_v, nullptr, nullptr, 0,
                         &seed, nullptr);
}

int gravac_threshold_compress(const float* grad, float* residual, int64_t n, float tau, int32_t* out_idx, float* out_val,
                              int64_t out_capacity, int64_t* out_count, double* out_stats, void* workspace,
                              size_t workspace_bytes, void* stream_v)
{
    if (!residual) return GRAVAC_ERR_INVALID_ARG;
    const double one = 1.0;
    return compress_impl(grad, residual, n, &one, 1, 0, nullptr, 0, out_idx, out_val, out_capacity, out_count, out_stats,
                         workspace, workspace_bytes, 0, (hipStream_t)stream_v, nullptr, nullptr, 0, nullptr, nullptr, &tau);
}

int gravac_recompress(const int32_t* idx1, const float* val1, int64_t k1, double cf_rel, const int64_t* seg_counts,
                      int n_seg, float* residual, int64_t n, int32_t* out_idx, float* out_val, int64_t out_capacity,
                      int64_t* out_count, double* out_stats, void* workspace, size_t workspace_bytes, unsigned flags,
                      void* stream_v)
{
    if (!idx1 || !val1 || k1 <= 0 || n_seg < 0 || (n_seg > 0 && !seg_counts)) return GRAVAC_ERR_INVALID_ARG;
    if (residual && (n <= 0 || n > 2147483647LL)) return GRAVAC_ERR_INVALID_ARG;
    std::vector<int64_t> off;
    if (n_seg > 0) {
        off.resize((size_t)n_seg + 1);
        off[0] = 0;
        for (int t = 0; t < n_seg; ++t) {
            if (seg_counts[t] <= 0 || seg_counts[t] > k1) return GRAVAC_ERR_INVALID_ARG;
            off[t + 1] = off[t] + seg_counts[t];
        }
        if (off[n_seg] != k1) return GRAVAC_ERR_INVALID_ARG;
    }
    return compress_impl(val1, nullptr, k1, &cf_rel, 1, 0, n_seg > 0 ? off.data() : nullptr, n_seg, out_idx, out_val,
                         out_capacity, out_count, out_stats, workspace, workspace_bytes, flags, (hipStream_t)stream_v,
                         idx1, residual, n, nullptr, nullptr);
}

int gravac_commit(const int32_t* idx, int64_t count, float* residual, int64_t n, void* stream_v)
{
    if (!residual || count < 0 || n <= 0 || n > 2147483647LL || (count > 0 && !idx)) return GRAVAC_ERR_INVALID_ARG;
    if (count == 0) return GRAVAC_OK;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(commit_kernel, dim3((uint32_t)blocks), dim3(256), 0, (hipStream_t)stream_v, idx, count, residual, n);
    if (hipGetLastError() != hipSuccess) return GRAVAC_ERR_HIP;
    return GRAVAC_OK;
}

int gravac_decompress_workspace_bytes(int W, int64_t n, size_t* bytes_out)
{
    if (!bytes_out || W < 1 || n <= 0 || n > 2147483647LL) return GRAVAC_ERR_INVALID_ARG;
    const int64_t ntile = (n + DTILE - 1) / DTILE;
    const int wn = W < DMAXW ? W : DMAXW;
    *bytes_out = align_up(sizeof(uint32_t) * (size_t)wn * (size_t)(ntile + 1), 256);
    return GRAVAC_OK;
}

// bounds: device memory for the tile boundaries of up to DMAXW messages (the caller's workspace or the library's static
// scratch, already checked for size), or null for the search path.
static int decompress_impl(const int32_t* idx, const float* val, const int64_t* counts, int W, int64_t n, float* dense_out,
                           float alpha, uint32_t* bounds, void* stream_v)
{
    hipStream_t stream = (hipStream_t)stream_v;
    if (!counts || !dense_out || W < 1 || n <= 0 || n > 2147483647LL) return GRAVAC_ERR_INVALID_ARG;
    int64_t total = 0;
    for (int w = 0; w < W; ++w) {
        if (counts[w] < 0) return GRAVAC_ERR_INVALID_ARG;
        total += counts[w];
    }
    if (total > 0 && (!idx || !val)) return GRAVAC_ERR_INVALID_ARG;
    if (total == 0) return GRAVAC_OK;
    const int64_t ntile = (n + DTILE - 1) / DTILE;
    const uint32_t grid = (uint32_t)(ntile < 1024 ? ntile : 1024);  // 4 workgroups (4 x 32 KiB LDS) on each of 256 CUs
    const bool plain = 4 * n > PLAIN_FROM && 4 * n <= PLAIN_BYTES;  // see store_tile
    int64_t at = 0;
    for (int w0 = 0; w0 < W; w0 += DMAXW) {
        const int wn = (W - w0 < DMAXW) ? W - w0 : DMAXW;
        WorkerOffsets wo;
        int64_t group = 0, longest = 0;
        for (int w = 0; w < wn; ++w) {
            wo.at[w] = at + group;
            group += counts[w0 + w];
            if (counts[w0 + w] > longest) longest = counts[w0 + w];
        }
        for (int w = wn; w <= DMAXW; ++w) wo.at[w] = at + group;
        at += group;
        if (group == 0) continue;
        if (bounds) {
            // tile boundaries of the group's messages first (the workspace is reused from group to group: stream order)
            const int bp = group < BROWS_PAIRS ? 1 : 4;
            const uint32_t pair_blocks = (uint32_t)((longest + 256 * bp - 1) / (256 * bp));
            hipLaunchKernelGGL(bp == 1 ? bounds_kernel<1> : bounds_kernel<4>, dim3(pair_blocks, (uint32_t)wn), dim3(256), 0,
                               stream, idx, wo, ntile, bounds);
            hipLaunchKernelGGL(plain ? decompress_ws_kernel<0> : decompress_ws_kernel<7>,
                               dim3(grid), dim3(256), 0, stream, idx, val, wo, wn, n, dense_out, (const uint32_t*)bounds, alpha);
        } else {
            hipLaunchKernelGGL(plain ? decompress_kernel<0> : decompress_kernel<DTILE / 1024>,
                               dim3(grid), dim3(256), 0, stream, idx, val, wo, wn, n, dense_out, alpha);
        }
    }
    if (hipGetLastError() != hipSuccess) return GRAVAC_ERR_HIP;
    return GRAVAC_OK;
}


int gravac_decompress_accumulate(const int32_t* idx, const float* val, const int64_t* counts, int W, int64_t n,
                                 float* dense_out, void* workspace, size_t workspace_bytes, void* stream_v)
{
    if (!counts || !dense_out || W < 1 || n <= 0 || n > 2147483647LL) return GRAVAC_ERR_INVALID_ARG;
    if (workspace) {
        size_t need = 0;
        if (gravac_decompress_workspace_bytes(W, n, &need) != GRAVAC_OK) return GRAVAC_ERR_INVALID_ARG;
        if (((uintptr_t)workspace & 255) || workspace_bytes < need) return GRAVAC_ERR_WORKSPACE;
    }
    return decompress_impl(idx, val, counts, W, n, dense_out, 1.0f, (uint32_t*)workspace, stream_v);
}

int gravac_decompress_update(const int32_t* idx, const float* val, const int64_t* counts, int W, int64_t n, float alpha,
                             float* params, void* workspace, size_t workspace_bytes, void* stream_v)
{
    if (!counts || !params || W < 1 || n <= 0 || n > 2147483647LL) return GRAVAC_ERR_INVALID_ARG;
    if (workspace) {
        size_t need = 0;
        if (gravac_decompress_workspace_bytes(W, n, &need) != GRAVAC_OK) return GRAVAC_ERR_INVALID_ARG;
        if (((uintptr_t)workspace & 255) || workspace_bytes < need) return GRAVAC_ERR_WORKSPACE;
    }
    return decompress_impl(idx, val, counts, W, n, params, alpha, (uint32_t*)workspace, stream_v);
}

int gravac_decompress_accumulate_static(const int32_t* idx, const float* val, const int64_t* counts, int W, int64_t n,
                                        float* dense_out, void* stream_v)
{
    if (!counts || !dense_out || W < 1 || n <= 0 || n > 2147483647LL) return GRAVAC_ERR_INVALID_ARG;
    size_t need = 0;
    if (gravac_decompress_workspace_bytes(W, n, &need) != GRAVAC_OK) return GRAVAC_ERR_INVALID_ARG;
    if (need > (size_t)GRAVAC_STATIC_SCRATCH_BYTES) return GRAVAC_ERR_STATIC_LIMIT;
    uint32_t* bounds = nullptr;
    if (const int rc = static_scratch(&bounds)) return rc;
    return decompress_impl(idx, val, counts, W, n, dense_out, 1.0f, bounds, stream_v);
}

int gravac_read_status(const void* workspace, void* stream_v, int32_t* out8)
{
    if (!workspace || !out8) return GRAVAC_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)stream_v;
    if (hipStreamSynchronize(stream) != hipSuccess) return GRAVAC_ERR_HIP;
    Status s;
    if (hipMemcpy(&s, workspace, sizeof(Status), hipMemcpyDeviceToHost) != hipSuccess) return GRAVAC_ERR_HIP;
    out8[0] = s.any_fail; out8[1] = s.n_fail; out8[2] = s.error; out8[3] = s.n_seg; out8[4] = s.n_narrow;
    out8[5] = s.n_wide;
    out8[6] = out8[7] = 0;
    return GRAVAC_OK;
}

const char* gravac_strerror(int code)
{
    switch (code) {
        case GRAVAC_OK: return "ok";
        case GRAVAC_ERR_INVALID_ARG: return "invalid argument";
        case GRAVAC_ERR_CAPACITY: return "output capacity too small";
        case GRAVAC_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case GRAVAC_ERR_HIP: return "HIP runtime error";
        case GRAVAC_ERR_STATIC_LIMIT: return "W and n exceed what the library's static scratch holds";
        case GRAVAC_ERR_CAPTURE: return "call cannot be recorded into a HIP graph (layerwise or profiled call on a capturing stream)";
        default: return "unknown error code";
    }
}

}  // extern "C"
