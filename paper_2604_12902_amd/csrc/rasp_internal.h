// rasp_internal.h -- structures shared by the host runtime and the kernels of
// librasp (never exposed through the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rasp {

constexpr int kWave = 64;              // CDNA wavefront width
constexpr int kMaxMulti = 64;          // batches per multi-batch launch
constexpr uint32_t kMaxMemWords = 1u << 30;
constexpr uint32_t kNoCap = 0xffffffffu;   // a persistent launch that is not a first pass

// Device view of one batch: struct-of-arrays machine state plus the packed
// per-machine shapes and the three word arenas (memory, tape, output), each
// machine's slice contiguous.  Memory slices start on 16-byte boundaries.
struct DevBatch {
    int32_t *i;
    int32_t *a;
    uint32_t *u0;
    uint32_t *y0;
    uint64_t *steps;
    uint8_t *status;
    uint32_t *n;
    uint32_t *ell;
    uint32_t *s;
    uint64_t *mem_off;                 // word offset of M_v in M
    uint64_t *t_off;                   // word offset of tape_v in T
    uint64_t *y_off;                   // word offset of y_v in Y
    // words of M_v at or above hw[v] are zero and not stored (c0's zero tail
    // before anything is written there); a multiple of 4, at most n_v
    // rounded up to 4, which means every word is stored
    uint32_t *hw;
    int32_t *M;
    int32_t *T;
    int32_t *Y;
    uint64_t N;
    uint32_t isa;
    uint32_t fresh;                    // 1: state is c0, built from the packed inputs below
    uint32_t wshift;                   // 32 - w: words are w-bit values, sign-extended
    uint32_t pad;
    const int32_t *prog;               // packed programs / inputs of a fresh batch
    const uint64_t *prog_off;
    const int32_t *tape;
    const uint64_t *tape_off;
};

// Table of batches advanced together by one launch.  Machine g of the launch
// is machine g - start[k] of batch k, for the k with start[k] <= g < start[k+1].
struct BatchTable {
    DevBatch b[kMaxMulti];
    uint64_t start[kMaxMulti + 1];
    uint32_t budget[kMaxMulti];        // transitions this launch may apply per machine
    uint32_t count;
    uint32_t pad;
};

// Counters of one persistent launch (device memory, zeroed by a fill kernel
// before every launch so that the launch can sit in a HIP graph).
struct QueueState {
    unsigned long long head;           // next unclaimed work item
    unsigned long long survivors;      // items appended to the survivor list
    unsigned long long retired;        // transitions retired (statistics)
    unsigned long long pad;
    unsigned long long misfits;        // hot-cell first pass: survivors whose hot cells do not all fit
    unsigned long long head_m;         // next unclaimed misfit
    unsigned long long pad2[2];
    unsigned long long count[10];       // traces: machines in each list,
    unsigned long long next[10];        // and the next unclaimed one
};

// Hot-cell tables.  A first pass profiles the last R transitions of every
// machine it leaves running: the 2-word cells (words 2x, 2x + 1) its
// fetches and data accesses touch.  A survivor whose cells can be placed in
// S slots without two sharing one (slot of cell x = bits [16, 16 + log2 S)
// of x * c, c chosen per machine) is a fit; the persistent kernel then keeps
// exactly those cells in LDS and every access of its steady loop is an LDS
// hit.  Fit p of the survivor list has multiplier mult[p] and cells
// tags[p S + s] (0xffff: empty slot); misfits go to a list of their own
// (count q->misfits), run with their memory in HBM by a second persistent
// launch beside the fits' launch, so that no wave mixes the two.
struct HotArgs {
    uint32_t S;                        // slots per machine (power of two, 8..64); 0: off
    uint32_t lgS;
    uint32_t R;                        // profiled transitions at the end of the first pass
    uint32_t bw;                       // profile bitmap words per lane
    uint32_t *mult;
    uint16_t *tags;
    uint32_t *mis;                     // misfit list
};

// Lists of machines (index in the launch, transitions to go) behind a first
// pass: what the trace kernel does with its survivors.
enum : uint32_t {
    kListFirst = 0,                    // the first pass's survivors (count in survivors)
    kListMisfit = 1,                   // a hot-cell first pass's misfits (count in misfits)
    kListWarm = 2,                     // survivors of a second pass, where the first was short
    kListGeneral = 3,                  // not for nodes: k_whole, or the work queue if they are many
    kListFull = 4,                     // need larger tables
    kListMain = 5,                     // run in nodes
    kListLast = 6,                     // of kListFull, not for nodes
    kListLate = 7,                     // of kListMain, seen late not to fit or to step in general often
    kListEnd = 8,                      // near the end of their budget
    kListDone = 9,                     // (no list: finished)
    kLists = 10
};
struct TraceArgs {
    uint32_t NO, ND;                   // nodes and data words a lane
    uint32_t in;                       // the list this launch works on
    // k_trace: where machines go that step in general too often, that fill
    // their tables too often, and (stop > 0) that have run `stop` transitions
    uint32_t often, full, rest, stop;
    uint32_t events, events_sh;        // how often: events general steps and one in 2^events_sh transitions
    uint32_t fulls, fulls_sh;
    uint32_t dense, least;             // machines a wave (0: as few as spread them over the launch), on `least` blocks at least
    uint32_t all;                      // k_whole: this many machines from the first one on, no list (0: list `in`),
    uint32_t few;                      // the longest list it takes,
    uint32_t spread;                   // the waves it spreads a short one over,
    uint32_t slab;                     // the bytes of LDS of each,
    uint32_t already;                  // and the first pass's transitions
    uint32_t *idx[9], *left[9];       // by list (left null: the budget less the first pass)
};
// Waves a block of k_trace (at most) and of k_whole.  One-wave blocks of a
// launch of a few waves a CU land on one SIMD of each (k_whole, a loop of four
// instructions: 143 ns a transition with 256 such blocks, 310 with 1,024); the
// waves of one block are spread.
constexpr uint32_t kTraceWpb = 8, kWholeWpb = 4;
constexpr uint32_t kTraceMax = 8;      // transitions of a node at most
constexpr uint32_t kTraceRounds = 16;  // general steps of a lane between runs of macro steps
constexpr uint32_t kTraceNear = 32;    // macro steps before its end from which a lane waits for others,
constexpr uint32_t kTraceEnd = 1;      // and from which its machine leaves
// Sorted survivors run kTraceSort transitions first, transients among them,
// which shows nearly all that do not run in small tables.  Meanwhile kSortEvents
// and kSortFulls stand for kTraceEvents and kTraceFulls (with those 24 and 2 at
// once fig1's 262,144 machines take 15.37 ms, not 15.55, plain-scale with 20,000
// transitions 3.26, not 3.39).
constexpr uint32_t kTraceSort = 512;
constexpr uint32_t kSortEvents = 64, kSortFulls = 4;
constexpr uint32_t kTraceEvents = 24, kTraceEventsSh = 11;   // general steps (and one in 2^Sh transitions) before a machine leaves
constexpr uint32_t kTraceFulls = 2, kTraceFullsSh = 10;      // times its tables are full before it leaves
// The same for kListLate, whose machines take a chain of k_whole from then on
// (with kTraceEvents' and kTraceFulls' numbers fig1 and beaver are the same
// within 1%, plain-scale 1-3% slower).
constexpr uint32_t kLateEvents = 64, kLateEventsSh = 8;
constexpr uint32_t kLateFulls = 16, kLateFullsSh = 9;
// Sorted survivors go to k_whole together from one in kJoinShare on that has to
// (k_join): plain-scale has one in 41, fig1 and beaver none in 2,800 and 67,000.
constexpr uint32_t kJoinShare = 64;
constexpr uint32_t kCrowdLeast = 8;    // machines of a wave from which on most of them may leave together,
constexpr uint32_t kCrowdEvents = 8, kCrowdRate = 16;        // with 8 general steps and one in 16 transitions (4 steps: the same times)
// Machines a wave of those beside the rest: few, since they compile often (fig1
// in tables of 48 nodes 11.6 ms with 4, 19.9 with 8; in the pass as it is now 4
// and 16 take 15.6 ms each).
constexpr uint32_t kTraceDense = 4;
constexpr uint32_t kTraceNodes = 16, kTraceData = 10;        // 7 waves a CU
constexpr uint32_t kTraceNodes2 = 48, kTraceData2 = 40;      // 2 waves a CU
// The largest memory traces are compiled for.  Positions would do to 2^15, but
// a program that sweeps a large array computes addresses anew on every round
// and ends up on the general lists, without a slot in LDS there (rollouts,
// n = 2,048: 159 ms with traces, 144 without).
constexpr uint32_t kTraceMaxN = 1u << 10;
constexpr uint32_t trace_lds_bytes(uint32_t NO, uint32_t ND) { return NO * (1024u + 128u) + (ND + 2u) * 256u + ND * 128u; }
constexpr uint32_t kWholeMaxN = 2048;  // largest memory k_whole takes (4 lanes a wave)
constexpr uint64_t kLdsGrain = 1280;   // LDS of a block is taken in units of this
constexpr uint64_t whole_lds_bytes(uint32_t max_n, uint32_t sh) { return (max_n + 2ull) << (sh + 2u); }
// A launch of k_whole: 2^sh lanes a wave, each wave with `slab` bytes of LDS,
// on `blocks` blocks; no blocks where the memories are too large for it.
struct WholeShape {
    uint32_t sh, slab, blocks;
};
constexpr WholeShape whole_shape(uint32_t max_n, uint64_t total, uint64_t lds, uint32_t cus)
{
    WholeShape w{6, 0, 0};
    if (max_n > kWholeMaxN) return w;
    while (w.sh > 2 && kWholeWpb * whole_lds_bytes(max_n, w.sh) > lds) --w.sh;
    const uint64_t slab = whole_lds_bytes(max_n, w.sh);
    const uint64_t block = (kWholeWpb * slab + kLdsGrain - 1) / kLdsGrain * kLdsGrain;
    const uint64_t per_cu = lds / block < 8 ? lds / block : 8, most = (total + kWholeWpb - 1) / kWholeWpb;
    w.slab = static_cast<uint32_t>(slab);
    w.blocks = static_cast<uint32_t>(most < per_cu * cus ? most : per_cu * cus);
    return w;
}

// Descriptor-check error bits.
enum : uint32_t {
    kErrOffsets = 1u,                  // prog_off / tape_off decreasing
    kErrProgTooLong = 2u,              // 2m > n
    kErrTapeTooLong = 4u,              // |x| > l
    kErrMemSize = 8u,                  // n == 0 or n > 2^30
    kErrStateRange = 16u,              // u0 > l or y0 > s in a loaded state
    kErrWordRange = 32u                // a word outside the w-bit range
};

struct LaunchShape {
    int cus;
    int lds_bytes;
};

// kernel launchers (rasp_kernels.hip)
// Layout of a batch from a device descriptor: n, l, s per machine (b.n,
// b.ell, b.s), the exclusive offsets b.mem_off (padded n), b.t_off, b.y_off,
// totals[0..3] = sums of padded n, l, s and n, err |= descriptor error bits,
// mx[0] = max n, mx[1] != 0 iff some n is not a power of two, mx[2] = max l.
// sums holds layout_scratch_words(N) words; mx and totals start at zero.
hipError_t launch_layout(const uint64_t *prog_off, const uint64_t *tape_off, const uint32_t *mem_words,
                         uint32_t def_mem, const uint32_t *tape_cap, const uint32_t *out_cap, uint32_t def_out,
                         uint64_t N, DevBatch b, uint64_t *sums, uint64_t *totals, uint32_t *err, uint32_t *mx,
                         hipStream_t st);
uint64_t layout_scratch_words(uint64_t N);
hipError_t launch_scan_u64(const uint64_t *in, uint64_t *out_excl, uint64_t N,
                           uint64_t *block_sums, uint64_t *total, hipStream_t st);
hipError_t launch_scan_u32(const uint32_t *in, uint64_t *out_excl, uint64_t N,
                           uint64_t *block_sums, uint64_t *total, hipStream_t st);
uint64_t scan_scratch_words(uint64_t N);
hipError_t launch_pack(DevBatch b, const int32_t *prog, const uint64_t *prog_off,
                       const int32_t *tape, const uint64_t *tape_off, hipStream_t st);
hipError_t launch_check_state(DevBatch b, uint32_t *err, hipStream_t st);  // u0, y0, and i, a when w < 32
hipError_t launch_probe(DevBatch b, hipStream_t st);
// wm: some batch of the launch has words narrower than 32 bits
hipError_t launch_plain(const BatchTable *tab, uint64_t total, uint32_t cap,
                        uint32_t isa, bool pow2, bool pack, bool wm, uint32_t *surv, QueueState *q,
                        hipStream_t st, const HotArgs *hot = nullptr);
// cap < UINT32_MAX with surv non-null: a first pass (machines still running
// after cap transitions are appended to surv, q->survivors counts them)
hipError_t launch_persistent(const BatchTable *tab, uint64_t total, const uint32_t *work,
                             uint32_t already, uint32_t isa, bool pow2, bool wm, uint32_t epoch,
                             uint32_t lds_words, uint32_t max_n, uint32_t max_ell,
                             uint32_t waves_per_block, uint32_t blocks, uint32_t cap, uint32_t *surv,
                             QueueState *q, hipStream_t st, uint32_t which = 0,
                             const uint32_t *rest_left = nullptr, uint32_t few = 0, uint32_t cus = 0);
// (which 1: the work list is a hot-cell first pass's misfit list, counted by
// q->misfits and claimed through q->head_m; kListGeneral, kListEnd: that
// list, rest_left its machines' transitions to go; a list of at most `few`
// machines is left alone, or with a cap one of more; cus: the compute units that
// the waves of a list with memories in HBM are spread over)
// sorted survivors' lists into one, kListGeneral, where `join` lanes hold them
// and some are there already
hipError_t launch_join(const TraceArgs &ta, QueueState *q, uint32_t join, hipStream_t st);
// whole memories in LDS, 2^sh lanes a wave, over list ta.in if it has at
// most ta.few machines
hipError_t launch_whole(const BatchTable *tab, uint32_t isa, bool pow2, bool wm, const TraceArgs &ta, uint32_t sh,
                        uint32_t blocks, QueueState *q, hipStream_t st);
// the trace kernel over list ta.in
hipError_t launch_trace(const BatchTable *tab, uint32_t already, uint32_t isa, bool wm, const TraceArgs &ta,
                        uint32_t wpb, uint32_t blocks, QueueState *q, hipStream_t st);
// the persistent kernel over the fits of a hot-cell first pass, each
// machine's hot cells in its lane's LDS table
hipError_t launch_persistent_hot(const BatchTable *tab, const uint32_t *work, uint32_t already, uint32_t isa,
                                 bool pow2, bool wm, uint32_t epoch, const HotArgs &hot,
                                 uint32_t waves_per_block, uint32_t blocks, QueueState *q, hipStream_t st);
// LDS words per lane of a hot-cell table of S slots (two words and a 16-bit
// cell tag per slot)
constexpr uint32_t hot_slot_words(uint32_t S) { return 2u * S + S / 2u; }
// profile bitmap words per lane for memories of at most max_n words
constexpr uint32_t hot_bitmap_words(uint32_t max_n) { return ((max_n + 1u) / 2u + 31u) / 32u; }
constexpr uint32_t kHotMaxN = 2048;     // largest memory a hot-cell launch profiles
// err |= kErrWordRange if some of the `count` words is not a w-bit value
hipError_t launch_check_words(const int32_t *w, uint64_t count, uint32_t wshift, uint32_t *err,
                              hipStream_t st);
// the same for words [off[0], off[N]) of w, the offsets in device memory
hipError_t launch_check_words_off(const int32_t *w, const uint64_t *off, uint64_t N, uint32_t wshift,
                                  uint32_t *err, hipStream_t st);
// LDS words of one lane's slot for a launch (memory words, four spare words
// and, when every memory fits and tapes are short, the tape); 0 for memory in HBM
uint32_t slot_words(uint32_t lds_words, uint32_t max_n, uint32_t max_ell);
constexpr uint32_t kTapeLdsMax = 64;     // tapes up to this many words are staged in LDS
hipError_t launch_zero_queue(QueueState *q, hipStream_t st);
hipError_t launch_reset_head(QueueState *q, hipStream_t st);     // head = 0, counts kept
void init_kernel_attributes();
hipError_t launch_running(const BatchTable *tab, uint64_t total, unsigned long long *counts,
                          hipStream_t st);
hipError_t launch_digest(DevBatch b, uint64_t *out, hipStream_t st);
// every machine's zero tail stored (zero_fill) or declared stored: hw = n rounded up to 4
hipError_t launch_tails(DevBatch b, bool zero_fill, hipStream_t st);
// per-machine scalars into device buffers (null pointers skipped)
hipError_t launch_fetch_scalars(DevBatch b, uint8_t *status, uint64_t *steps, int32_t *i, int32_t *a,
                                uint32_t *u0, uint32_t *y0, hipStream_t st);
hipError_t launch_steps_sum(DevBatch b, unsigned long long *out, hipStream_t st);
hipError_t launch_gather_words(const int32_t *src, const uint64_t *off, const uint32_t *len,
                               uint64_t N, int32_t *dst, const uint64_t *dst_off,
                               hipStream_t st);
hipError_t launch_scatter_words(const int32_t *src, const uint64_t *src_off,
                                const uint32_t *len, uint64_t N, int32_t *dst,
                                const uint64_t *dst_off, hipStream_t st);

}  // namespace rasp
