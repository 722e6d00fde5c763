// The search kernel: one 1024-thread workgroup per utterance loops over every
// decoded frame of its utterance (token passing, Sec. 3; the per-frame
// Viterbi beam search of Alg. 1).
//
// Frame k (token set S_k) in one workgroup:
//   1. expansion of the emitting arcs of S_{k-1}: each wave takes two chunks
//      of 64 consecutive arcs of the set at a time, finds their tokens from
//      the set's emitting-arc prefix and issues all their loads together; the
//      frame's log-likelihood row sits in LDS.  The frame's tokens live in a
//      hash table in LDS (state -> cost key); recombination is an LDS 32-bit
//      atomicMin on the ordered cost key, the first touch of a state appends
//      its slot to a slot list and fetches the state's line of the graph
//      ahead of its use in steps 4 and 1;
//   2. epsilon closure: a lowered token whose state has epsilon arcs becomes
//      an item of its wave's own queue, drained without a barrier: an item
//      whose state has a closure list offers its paths, spread over the wave,
//      the others their arcs one by one.  What does not fit the queue goes to
//      a device-memory list that the whole workgroup relaxes after a barrier.
//      (One list of the workgroup's items, its paths dealt evenly to the waves
//      after a barrier, was slower everywhere: 256 utterances 62.6 ms against
//      58.8, one 17.6 against 17.1);
//   3. pruning: beam limit from the frame's best cost key and, when more
//      tokens lie within it than max_active, the exact max_active-th
//      smallest key by radix select over an LDS histogram;
//   4. compaction of the survivors into S_k (device memory, and LDS for the
//      next expansion), with the prefix of their emitting out-degrees, and
//      the set's lattice record regions; the table's slots are cleared as
//      they are read.
// Back-pointers and lattice records need nothing the next frame needs: the
// record kernel derives them afterwards from the stored token sets, every
// frame of every utterance in parallel (a token's back-pointer is the lowest
// arc whose candidate cost equals the token's cost, which is what a minimum
// over (cost, arc) pairs would have kept), so the search keeps costs only
// and writes nothing per candidate.
//
// Three token tables, one template: a small one in LDS beside the previous
// set and the log-likelihood row (kSmall), one of twice the slots that takes
// their place in LDS while the sets are too large for that copy (kBig; the
// set and the row are then read from device memory), and one in device memory
// (kDev; the row and a larger copy of the set have the LDS to themselves).
// A frame that reaches more states than its table holds is redone on
// the next larger one.  Every table is private to its workgroup and there are
// no per-frame launches; the only device-scope synchronisation is the
// search's progress count, published every pub_k token sets when record
// workgroups (below) or the incremental lattice pass follow it.
//
// Barriers of a frame: after step 2 and after step 4, and those of the spilled
// items' rounds and of the selection when there are any.  The frame's counters
// have two copies by frame parity; the other copy is cleared between the two
// barriers, when every wave has left the frame before, so that a frame begins
// without a barrier of its own.
//
// What bounds a frame: the chain of its dependent accesses, since one
// workgroup cannot be split over CUs without a device-wide barrier per step
// (about 1 us each).  The chain is state record -> arcs -> log-likelihood and
// table -> closure list; three of its links miss the L2 (0.8-1 us each), the
// rest is LDS round trips (about 130 clocks) and barriers.  Hence the LDS
// table, the chunk descriptions instead of a search for each arc's token, the
// next row and the claimed states' lines fetched without registers, and two
// barriers a frame.  Measured per frame, one utterance of the 25M-arc graph
// (about 1000 tokens): 14.5 -> 14.0 us (compaction 4.3 -> 1.9, the expansion
// takes over part of its misses); about 20 tokens: 4.1 -> 3.3 us; frames of
// about 4000 tokens, most of which the small table could not hold and redid in
// device memory: 120 -> 92 us with the big LDS table; frames of about 7,200
// tokens on the device-memory table: 264 -> 208 us with the row, the set and
// its chunks in LDS (247 with the row and sets of up to 2944 tokens only); a
// decode of 500 frames of up to 7000 tokens, a few of them on that table: 48.0
// -> 43.0 ms.
//
// This header is compiled twice, once per translation unit:
// search_kernel.hip instantiates the search alone, search_record_kernel.hip
// the search with record workgroups appended to its launch.
#pragma once

#include <cstddef>
#include <type_traits>

#include "device_util.h"
#include "record_set.h"

namespace wfd {

namespace {

constexpr int kT = 1024;                  // threads per workgroup
constexpr int kW = kT / kWave;            // waves per workgroup
// token tables
constexpr int kSmall = 0, kBig = 1, kDev = 2;
constexpr int kSlotBits = 13;
constexpr int kSlots = 1 << kSlotBits;    // slots of the small LDS table
constexpr int kFill = 6144;               // states per frame it takes
constexpr int kBigBits = 14;
constexpr int kBigSlots = 1 << kBigBits;  // slots of the big LDS table
constexpr int kBigFill = 12800;           // states per frame it takes
constexpr int kSetCache = 2496;           // tokens of the previous set kept in LDS for the expansion
constexpr int kDevSet = 12160;            // the same beside the device-memory table
constexpr int kCs = 512;                  // 64-arc chunks of the previous set described in LDS
constexpr int kDevCs = 1024;              // the same beside the device-memory table
constexpr int kQueue = 128;               // epsilon items per wave queue
constexpr int kChunks = 2;                // 64-arc or 64-path chunks a wave has in flight (as pin() is called)
constexpr int kMaxProbe = 64;             // linear-probe bound (the fill limit keeps probes short)
constexpr int kOverflow = 1;              // frame result: the table filled up
constexpr uint32_t kNoKey = 0xFFFFFFFEu;   // a key no state has (state ids are below 2^31)
constexpr int kRowMax = 6144;             // log-likelihood columns a frame's LDS row holds
constexpr uint32_t kClosureSizeMask = (1u << kClosureSizeBits) - 1u;

static_assert(kHistBins <= 2 * kW * kQueue, "the select histogram aliases the epsilon queues");
static_assert(kCs <= kDevCs && kDevCs <= kW * kWave, "a wave's chunk descriptions fit its lanes");

// One frame's counters, two copies by frame parity.
struct Cnt {
    uint32_t best;             // smallest cost key among the frame's tokens
    int overflow;              // more states than the table's fill limit
    unsigned long long alloc;  // emitting degrees << 32 | survivors placed
    unsigned long long xsum;   // survivors without emitting arcs << 32 | epsilon degrees of the survivors
    int nslots;                // claimed slots
    int cnt;                   // tokens within the beam
    int spill_n[2];            // epsilon items in the device-memory lists
};

__device__ __forceinline__ Cnt empty_cnt() { return Cnt{kEmptyKey, 0, 0ull, 0ull, 0, 0, {0, 0}}; }

struct Sh {
    Cnt c[2];
    int status;                // sticky error of the utterance
    int bin, before;
    int scan[20];
    uint32_t sink[kWave];      // where fetched-ahead words land, never read
};

// Running values of the utterance, thread 0's own (in LDS: no registers held).
struct Run {
    int64_t le, lx;      // emitting and epsilon regions reserved so far (le: the arcs expanded, too)
    int64_t eps;         // epsilon out-arcs of the survivors
};

// Profiling counters, kept by thread 0 in LDS (in registers they would
// take space in every thread).
struct Prof {
    unsigned long long ph[7];    // device clock ticks per step
    unsigned long long cur[4];   // the current frame's steps
    unsigned long long t_last;
    unsigned long long t_sub;
};

// What lies in LDS beside the small table, with the big one, and with the
// device-memory table (the row in the same place as beside the small table).
struct SmallLds {
    float row[kRowMax];            // the frame's log-likelihood row (L <= kRowMax)
    float2 cb[kSetCache];          // the last token set: cost, first emitting record - epre (as int)
    int32_t epre[kSetCache];       // and the prefix of its emitting degrees
    uint16_t slots[kFill];
    uint32_t keys[kSlots];
    uint32_t vals[kSlots];
};

struct BigLds {
    uint32_t keys[kBigSlots];
    uint32_t vals[kBigSlots];
};

struct DevLds {
    float row[kRowMax];
    float2 cb[kDevSet];
    uint2 am[kDevCs];              // the chunk descriptions of a larger set
    uint16_t cs[kDevCs];
};

struct Lds {
    Sh sh;
    Prof pf;
    Run run;
    UttLayout ly;                      // the utterance's layout (in LDS: no registers held for it)
    // The 64-arc chunks of the last set: the token owning a chunk's first
    // arc, and a mask with bit i - 1 set where arc i of the chunk (1-63) is
    // the first of its token.  Every token has an arc, so the token owning
    // arc i is the first one plus the mask's bits below i.
    uint2 am[kCs];
    uint16_t cs[kCs];
    uint2 wq[kW * kQueue];             // the waves' epsilon queues, or the select histogram
    uint32_t wql[kW * kQueue];         // the queue items' closure words
    union {
        SmallLds s;
        BigLds b;
        DevLds d;
    };
};
static_assert(offsetof(SmallLds, row) == offsetof(DevLds, row), "one place for the row");
// (a fetch's LDS address has 16 bits; the kernel's Lds lies at 0 unless it
// gets another shared variable, which would be small)
static_assert(offsetof(Lds, s.row) + sizeof(SmallLds::row) <= 63 * 1024, "a row fetch reaches the whole row");

// Where the chunks are described beside table M, and how many.
template <int M>
__device__ __forceinline__ uint2 *chunk_am(Lds &lds)
{
    if constexpr (M == kDev) return lds.d.am;
    else return lds.am;
}

template <int M>
__device__ __forceinline__ uint16_t *chunk_cs(Lds &lds)
{
    if constexpr (M == kDev) return lds.d.cs;
    else return lds.cs;
}

template <int M>
constexpr int kChunksMax = M == kDev ? kDevCs : kCs;
static_assert(sizeof(Lds) <= 160 * 1024, "the workgroup's LDS");

// Fetch one word per active lane into LDS at `to` + 4 * lane (the same `to` in
// every lane) without a register or a wait: to bring its cache line near (into
// Sh::sink, which nobody reads), or with a later fetch_wait and barrier to fill
// an array.  (m0, the fetch's LDS address, is put back: it is the compiler's.)
__device__ __forceinline__ void fetch_lds(const void *ptr, const void *to)
{
    // (the low half of a pointer to LDS is the LDS address)
    const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(to));
    uint32_t keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep)
                 : "v"(ptr), "s"(at)
                 : "memory");
}

// The wave's fetches so far have arrived (the compiler does not count them).
__device__ __forceinline__ void fetch_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Table loads: plain in LDS; in device memory they bypass the CU's L1, since
// the table's atomics are performed in L2.
template <int M, typename T>
__device__ __forceinline__ T tld(const T *ptr)
{
    if constexpr (M == kDev)
        return __hip_atomic_load(const_cast<T *>(ptr), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        return *ptr;
}

// With the slot list (and the table) in device memory their own stores need
// the full barrier.
template <int M>
__device__ __forceinline__ void frame_barrier()
{
    if constexpr (M == kSmall) lds_barrier();
    else block_sync_vm();
}

// Token table of one frame: keys = state (kEmptyKey if free), vals = the
// ordered cost key of the state's token (kEmptyKey if none).  `slots` lists
// the claimed slots in claim order.
template <int M>
struct Tab {
    using Slot = typename std::conditional<M == kSmall, uint16_t, int32_t>::type;
    uint32_t *keys;
    uint32_t *vals;
    Slot *slots;
    uint32_t nslots;   // of the table (a power of two)
    int fill;
    int shift;         // 32 - log2(slots)
    uint32_t mul;      // hash multiplier
    __device__ __forceinline__ uint32_t first(uint32_t d) const
    {
        return hash_state(d, mul) >> shift;
    }
    __device__ __forceinline__ uint32_t next(uint32_t h) const { return (h + 1) & (nslots - 1u); }
};

// Mark that token `idx` begins at position st of the set's arcs and holds
// cn >= 1 of them, in the chunk descriptions b (first token) and m (begins)
// of n 64-arc chunks.  Each chunk's first arc has one owner; the masks are
// cleared by the wave that reads them.
__device__ __forceinline__ void mark_begin(uint16_t *b, uint2 *m, int n, int st, int cn, int idx)
{
    const int off = st & (kWave - 1);
    if (off != 0 && st < n * kWave)
        atomicOr(reinterpret_cast<uint32_t *>(m) + 2 * (st / kWave) + (off - 1) / 32, 1u << ((off - 1) & 31));
    int ch = (st + kWave - 1) / kWave;
    if (ch * kWave < st + cn && ch < n) {
        b[ch] = static_cast<uint16_t>(idx);
        for (ch++; ch * kWave < st + cn && ch < n; ch++) b[ch] = static_cast<uint16_t>(idx);
    }
}

// A wave's chunk descriptions, chunk wid + kW * lane of `nch` (from the end
// with `rev`) in each lane; the masks are cleared for their next use.
struct Chunks {
    int b;
    uint32_t lo, hi;
};

__device__ __forceinline__ Chunks take_chunks(const uint16_t *b, uint2 *m, int nch, int wid, bool rev)
{
    Chunks c{0, 0u, 0u};
    const int i = wid + kW * lane_id();
    if (i < nch) {
        const int ch = rev ? nch - 1 - i : i;
        c.b = b[ch];
        const uint2 x = m[ch];
        c.lo = x.x;
        c.hi = x.y;
        m[ch] = make_uint2(0u, 0u);
    }
    return c;
}

// The token owning this lane's arc of the wave's i-th chunk.
__device__ __forceinline__ int chunk_owner(const Chunks &c, int i)
{
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(c.lo), i);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(c.hi), i);
    const uint32_t b = __builtin_amdgcn_readlane(c.b, i);
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, b)));
}

// The values of several loads are used from here on: all of the loads are
// issued before the first wait (the compiler would else now and then move
// one, or part of one, behind the wait for another, or under the condition
// of its use: a round trip more).
__device__ __forceinline__ void pin(int4 &a, int4 &b)
{
    asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w));
}

__device__ __forceinline__ void pin(int4 &a, int4 &b, int4 &c, int4 &d)
{
    asm volatile(""
                 : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w), "+v"(c.x),
                   "+v"(c.y), "+v"(c.z), "+v"(c.w), "+v"(d.x), "+v"(d.y), "+v"(d.z), "+v"(d.w));
}

// Profiling: thread 0 adds the device clock since the previous mark to step
// i of the current frame (0-3), or to the time between frames (5).  A frame
// that is completed adds its steps to the totals; one abandoned for a larger
// table adds them to slot 6.
__device__ __forceinline__ void phase_mark(const Params &p, Prof &pf, int i)
{
    if (p.profile && threadIdx.x == 0) {
        const unsigned long long t = wall_clock64();
        if (i == 5) pf.ph[5] += t - pf.t_last;
        else pf.cur[i] += t - pf.t_last;
        pf.t_last = t;
    }
}

__device__ __forceinline__ void phase_fold(const Params &p, Prof &pf, bool done)
{
    if (p.profile && threadIdx.x == 0) {
        for (int i = 0; i < 4; i++) {
            pf.ph[done ? i : 6] += pf.cur[i];
            pf.cur[i] = 0;
        }
    }
}

// Profiling of a part of a step as thread 0 sees it: open, then close into
// slot i.
__device__ __forceinline__ void sub_open(const Params &p, Prof &pf)
{
    if (p.profile && threadIdx.x == 0) pf.t_sub = wall_clock64();
}

__device__ __forceinline__ void sub_close(const Params &p, Prof &pf, int i)
{
    if (p.profile && threadIdx.x == 0) pf.ph[i] += wall_clock64() - pf.t_sub;
}

// A wave's own epsilon work: an LDS queue of (table slot, cost bits) items
// with the closure word of each item's state (0 if not known), and the
// device-memory list that takes what does not fit (without closure words).
struct WaveQ {
    uint2 *q;        // this wave's LDS queue
    uint32_t *ql;    // the items' closure words
    int n;           // items in it (the same in every lane)
    int qcap;        // its capacity
    uint2 *spill;    // device-memory list of the current round
    int *spill_n;    // its LDS counter
    int scap;        // its capacity
};

// Lanes of `push` into the wave's queue, or into the device-memory list.
__device__ __forceinline__ void queue_push(Sh &sh, WaveQ &wq, bool push, int slot, float cand, uint32_t cl)
{
    const uint64_t m = __ballot(push);
    if (!m) return;
    if (push) {
        const int idx = wq.n + rank_in(m);
        const uint2 it = make_uint2(static_cast<uint32_t>(slot), __float_as_uint(cand));
        if (idx < wq.qcap) {
            wq.q[idx] = it;
            wq.ql[idx] = cl;
        } else {
            const int gi = atomicAdd(wq.spill_n, 1);
            if (gi < wq.scap) wq.spill[gi] = it;
            else sh.status = WFST_ECAPACITY;
        }
    }
    wq.n = min(wq.n + __popcll(m), wq.qcap);
}

// Offer R candidate costs per lane (act[r]) to the table.  The R offers go
// through each step together, so that their LDS atomics are in flight at the
// same time.  Called by the whole wave.
template <int M, int R, bool PUSH>
__device__ __forceinline__ void offer(const Params &p, const Tab<M> &t, Sh &sh, Cnt &c, WaveQ &wq,
                                      const bool *act, const uint32_t *d, const bool *d_eps, const uint32_t *cl,
                                      const float *cand, const uint32_t *key)
{
    const int lane = lane_id();
    // slot of each state: a compare-and-swap on the key claims a free slot
    // or finds the state's own, probing linearly on a collision
    uint32_t h[R], k[R];
#pragma unroll
    for (int r = 0; r < R; r++) h[r] = t.first(d[r]);
    if constexpr (M != kDev) {
        // In LDS every lane issues its compare-and-swap, so that the R
        // atomics of the wave are in flight together instead of one branch
        // (and one wait) each: an inactive lane compares and swaps a key no
        // state has, at a slot of its own, which changes nothing.
#pragma unroll
        for (int r = 0; r < R; r++) {
            const uint32_t at = act[r] ? h[r] : static_cast<uint32_t>(lane);
            k[r] = atomicCAS(t.keys + at, act[r] ? kEmptyKey : kNoKey, act[r] ? d[r] : kNoKey);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) k[r] = act[r] ? atomicCAS(t.keys + h[r], kEmptyKey, d[r]) : 0u;
    }
    // collisions: the lanes of all R offers that still need a slot probe on together
    bool over = false;
    for (int probe = 1;; probe++) {
        bool need[R], any = false;
#pragma unroll
        for (int r = 0; r < R; r++) {
            need[r] = act[r] && k[r] != kEmptyKey && k[r] != d[r];
            any = any || need[r];
        }
        if (!__ballot(any)) break;
        if (probe == kMaxProbe) {
            over = any;
            break;
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (need[r]) {
                h[r] = t.next(h[r]);
                k[r] = atomicCAS(t.keys + h[r], kEmptyKey, d[r]);
            }
        }
    }
    bool has[R], claimed[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        has[r] = act[r] && (k[r] == kEmptyKey || k[r] == d[r]);
        claimed[r] = act[r] && k[r] == kEmptyKey;
    }
    // recombination: the unsigned minimum of the cost keys (in LDS without a
    // branch: a lane without a slot takes the minimum of a slot of its own
    // and the empty key, which changes nothing)
    uint32_t old[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        if constexpr (M != kDev) {
            const uint32_t at = has[r] ? h[r] : static_cast<uint32_t>(lane);
            old[r] = atomicMin(t.vals + at, has[r] ? key[r] : kEmptyKey);
        } else {
            old[r] = has[r] ? atomicMin(t.vals + h[r], key[r]) : 0u;
        }
    }
    // newly claimed slots join the slot list, one LDS add per wave; their
    // states' lines are fetched ahead: the compaction reads the state record
    // and the next expansion the arcs behind it
    uint64_t mc[R];
    int pc[R], nc = 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        mc[r] = __ballot(claimed[r]);
        pc[r] = nc;
        nc += __popcll(mc[r]);
    }
    if (nc) {
        int b = 0;
        if (lane == 0) b = atomicAdd(&c.nslots, nc);
#pragma unroll
        for (int r = 0; r < R; r++)
            if (p.ahead && claimed[r]) fetch_lds(p.g.srec + d[r], sh.sink);
        b = __builtin_amdgcn_readlane(b, 0);
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (claimed[r]) {
                const int idx = b + pc[r] + rank_in(mc[r]);
                if (idx < t.fill) t.slots[idx] = static_cast<typename Tab<M>::Slot>(h[r]);
                else over = true;
            }
        }
    }
    if (over) c.overflow = 1;
    if constexpr (!PUSH) return;   // (the closure list that lowered the tokens holds their paths too)
    // lowered tokens whose state has epsilon out-arcs
#pragma unroll
    for (int r = 0; r < R; r++)
        queue_push(sh, wq, has[r] && key[r] < old[r] && d_eps[r], static_cast<int>(h[r]), cand[r], cl[r]);
}

// One candidate per lane.
template <int M>
__device__ __forceinline__ void offer1(const Params &p, const Tab<M> &t, Sh &sh, Cnt &c, WaveQ &wq,
                                       bool act, uint32_t d, bool d_eps, uint32_t cl, float cand, uint32_t key)
{
    offer<M, 1, true>(p, t, sh, c, wq, &act, &d, &d_eps, &cl, &cand, &key);
}

// Bin holding the rank-th smallest (1-based) of a histogram: sets sh.bin and
// sh.before (the count in lower bins).
__device__ __forceinline__ void select_bin(const uint32_t *h, int nbins, int rank, Sh &sh)
{
    const int per = (nbins + kT - 1) / kT;
    const int b0 = threadIdx.x * per;
    int local = 0;
    for (int i = 0; i < per; i++)
        if (b0 + i < nbins) local += static_cast<int>(h[b0 + i]);
    int total;
    const int excl = block_excl_scan(local, sh.scan, &total);
    if (rank > excl && rank <= excl + local) {
        int cum = excl;
        for (int i = 0; i < per && b0 + i < nbins; i++) {
            const int c = static_cast<int>(h[b0 + i]);
            if (rank <= cum + c) {
                sh.bin = b0 + i;
                sh.before = cum;
                break;
            }
            cum += c;
        }
    }
    __syncthreads();
}

// Shift of the first radix digit so that (lim - kb) >> shift fits the histogram.
__device__ __forceinline__ int first_shift(uint32_t kb, uint32_t lim)
{
    const uint32_t span = lim - kb;
    const int nb = span ? 32 - __clz(static_cast<int>(span)) : 0;
    return nb > kHistBits ? nb - kHistBits : 0;
}

// S_{k-1} for the expansion: beside the small table in LDS, beside the
// device-memory one in LDS if it fits there, else in device memory.
struct SetView {
    const float2 *cb;        // cost, first emitting record - epre
    const int32_t *epre;
    const int32_t *state;    // device memory (a set without cb)
    const uint32_t *key;
    const uint16_t *cs;      // chunk descriptions
    uint2 *am;
    int n;                   // tokens
    int a;                   // emitting out-arcs
};

// The token owning each lane's arc of the chunk at a0 without chunk
// descriptions: a 64-ary search for the first one, then the 64 tokens from it
// (every token has an arc) marked on the lanes.
__device__ __forceinline__ int window_owner(const int32_t *epre, int n, int a, int a0)
{
    const int t0 = search_le(epre, n, a0);
    const int tt = t0 + lane_id();
    const int pre = tt < n ? epre[tt] : 0x7FFFFFFF;
    const int nx = tt + 1 < n ? epre[tt + 1] : (tt < n ? a : 0x7FFFFFFF);
    return min(t0 + owner_scan(pre, nx - pre, a0), n - 1);
}

// The same for a set in device memory: the cost of each lane's token and its
// first emitting record - epre, the window's own loaded with its prefix (a
// gather by owner would be a round trip more).
__device__ __forceinline__ void window_token(const SetView &v, int a0, float &cst, int &rel)
{
    const int t0 = search_le(v.epre, v.n, a0);
    const int i = min(t0 + lane_id(), v.n - 1);
    const int pre = v.epre[i];
    const int nx = i + 1 < v.n ? v.epre[i + 1] : v.a;
    const int st = v.state[i];
    const uint32_t key = v.key[i];
    const bool in = t0 + lane_id() < v.n;
    const int o = min(owner_scan(in ? pre : 0x7FFFFFFF, in ? nx - pre : 0, a0), v.n - 1 - t0);
    cst = __shfl(okey_val(key), o, kWave);
    rel = __shfl(st + 2 - pre, o, kWave);
}

// Emitting expansion of S_{k-1} into the table (step 1).  The frame's
// log-likelihood row is read from LDS (srow) when it fits there, else, and with
// the big table, from device memory (grow).  kCb: the set has v.cb.
template <int M, bool kCb>
__device__ __forceinline__ void expand(const Params &p, const Tab<M> &t, Sh &sh, Cnt &c, const SetView &v,
                                       const float *srow, const float *grow, WaveQ &wq)
{
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const bool row_lds = M != kBig && p.L <= kRowMax;
    const int nch = (v.a + kWave - 1) / kWave;
    const bool described = kCb && nch <= kChunksMax<M>;
    const Chunks cd = take_chunks(v.cs, v.am, min(nch, kChunksMax<M>), wid, p.reverse != 0 && described);
    // wave w takes chunks w, w + kW, w + 2 kW, ... : every wave gets work
    int i = 0;   // chunks taken
    for (int c0 = wid; c0 < nch; c0 += kW * kChunks, i += kChunks) {
        // (this frame's cheapest candidate so far, and whether it is to be redone anyway)
        const uint32_t cur = c.best;
        if (__builtin_amdgcn_readfirstlane(c.overflow)) break;
        int a[kChunks], tk[kChunks], at[kChunks];
        float cst[kChunks];
        bool ok[kChunks];
#pragma unroll
        for (int r = 0; r < kChunks; r++) {
            // (a chunk past the end repeats the last one, with no lane active)
            const int ch = min(c0 + r * kW, nch - 1);
            const int a0 = (p.reverse ? nch - 1 - ch : ch) * kWave;
            a[r] = a0 + lane;
            ok[r] = c0 + r * kW < nch && a[r] < v.a;
            if constexpr (kCb) {
                if (described) tk[r] = chunk_owner(cd, i + r);
                else tk[r] = window_owner(v.epre, v.n, v.a, a0);
            } else {
                window_token(v, a0, cst[r], at[r]);
                at[r] += a[r];
            }
        }
        if constexpr (kCb) {
            float2 x[kChunks];
#pragma unroll
            for (int r = 0; r < kChunks; r++) x[r] = v.cb[tk[r]];
#pragma unroll
            for (int r = 0; r < kChunks; r++) {
                cst[r] = x[r].x;
                at[r] = __float_as_int(x[r].y) + a[r];
            }
        }
        int4 rec[kChunks];
#pragma unroll
        for (int r = 0; r < kChunks; r++) rec[r] = p.g.earc[ok[r] ? at[r] : 0];
        pin(rec[0], rec[1]);
        float lv[kChunks];
        if (row_lds) {
#pragma unroll
            for (int r = 0; r < kChunks; r++) lv[r] = srow[ok[r] ? rec[r].y : 0];
        } else {
#pragma unroll
            for (int r = 0; r < kChunks; r++) lv[r] = ldg(grow + (ok[r] ? rec[r].y : 0));
        }
        bool act[kChunks], de[kChunks];
        uint32_t d[kChunks], key[kChunks], cw[kChunks];
        float cnd[kChunks];
        uint32_t km = kEmptyKey;
#pragma unroll
        for (int r = 0; r < kChunks; r++) {
            const float t1 = cst[r] + __int_as_float(rec[r].z);
            cnd[r] = t1 - lv[r];
            key[r] = ok[r] ? okey(cnd[r]) : kEmptyKey;
            km = min(km, key[r]);
            d[r] = static_cast<uint32_t>(rec[r].x) & kDstMask;
            de[r] = rec[r].x < 0;
            cw[r] = static_cast<uint32_t>(rec[r].w);
        }
        // The batch's own cheapest candidate tightens the early-drop bound; it
        // is within that bound itself, so it is offered and the frame's best
        // key may take its value now.
        km = wave_min_u32(km);
        if (km < cur && lane == 0) atomicMin(&c.best, km);
        // (never +inf: a placeholder would claim a slot)
        const uint32_t bnd = min(drop_bound(km < cur ? km : cur, p.beam), kMaxKey);
#pragma unroll
        for (int r = 0; r < kChunks; r++) act[r] = ok[r] && key[r] <= bnd;
        offer<M, kChunks, true>(p, t, sh, c, wq, act, d, de, cw, cnd, key);
    }
}

// A closure entry's path cost: the cost of its item plus the path's weights
// one at a time in path order, which is the arithmetic of relaxing the path
// arc by arc.  Weights the path does not have are -0, which changes no sum.
__device__ __forceinline__ float path_cost(float c, const int4 &e0, const int4 &e1)
{
    c += __int_as_float(e0.y);
    c += __int_as_float(e0.z);
    c += __int_as_float(e0.w);
    c += __int_as_float(e1.x);
    c += __int_as_float(e1.y);
    c += __int_as_float(e1.z);
    c += __int_as_float(e1.w);
    return c;
}

// Offer R closure paths per lane: entry e[r] of the table for an item of cost
// cst[r] (live[r]).  The entry holds every path of up to seven arcs whole in
// its first two words; the third is loaded when some path of the wave is longer.
template <int M, int R>
__device__ __forceinline__ void offer_paths(const Params &p, const Tab<M> &t, Sh &sh, Cnt &c, WaveQ &wq,
                                            const bool *live, const int *e, const float *cst,
                                            uint32_t bnd)
{
    int4 e0[R], e1[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int4 *x = p.g.ctab + kClosureStride * static_cast<int64_t>(live[r] ? e[r] : 0);
        e0[r] = x[0];
        e1[r] = x[1];
    }
    if constexpr (R == 2) pin(e0[0], e1[0], e0[1], e1[1]);
    else pin(e0[0], e1[0]);
    bool act[R], de[R], longer = false;
    uint32_t d[R], key[R], cw[R];
    float cnd[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        cnd[r] = path_cost(cst[r], e0[r], e1[r]);
        longer = longer || (live[r] && e0[r].x < 0);
    }
    if (__ballot(longer)) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (live[r] && e0[r].x < 0) {
                const int4 e2 = p.g.ctab[kClosureStride * static_cast<int64_t>(e[r]) + 2];
                cnd[r] += __int_as_float(e2.x);
                cnd[r] += __int_as_float(e2.y);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        d[r] = static_cast<uint32_t>(e0[r].x) & kDstMask;
        de[r] = false;
        cw[r] = 0u;
        key[r] = okey(cnd[r]);
        act[r] = live[r] && key[r] <= bnd;
    }
    offer<M, R, false>(p, t, sh, c, wq, act, d, de, cw, cnd, key);
}

// Relax the epsilon arcs of one item per lane (valid) of the wave's queue or
// of the device-memory list: the item's state still holding the item's cost,
// i.e. no cheaper item of it follows.  A state with a closure list offers its
// paths, spread over the wave; a state without one relaxes its own arcs, and
// lowered tokens of states with epsilon arcs become items of the wave's queue.
// An item that comes with its state's closure word (icl) goes to the list
// without loading the state record.
template <int M>
__device__ __forceinline__ void relax(const Params &p, const Tab<M> &t, Sh &sh, Cnt &c, WaveQ &wq,
                                      bool valid, uint2 it, uint32_t icl)
{
    const int lane = lane_id();
    int xb = 0, xd = 0, cb = 0, cn = 0;
    bool first = false;
    int4 x0 = make_int4(0, 0, 0, 0);
    const float cst = __uint_as_float(it.y);
    const uint32_t bnd = drop_bound(c.best, p.beam);
    if (valid) {
        const uint32_t now = tld<M>(t.vals + it.x);
        if (okey(cst) == now && now <= bnd) {
            if (icl) {
                cb = static_cast<int>(icl >> kClosureSizeBits) - 1;
                cn = static_cast<int>(icl & kClosureSizeMask) + 1;
            } else {
                const int64_t s = static_cast<int64_t>(tld<M>(t.keys + it.x));
                const int4 lo = p.g.srec[s];
                x0 = p.g.srec[s + 1];
                const uint32_t cl = static_cast<uint32_t>(x0.w);
                // A list of one path is the state's only epsilon arc, into
                // a state without epsilon arcs: the copy of that arc in the
                // state record offers it below without loading the list.
                if (cl && (cl & kClosureSizeMask) != 0u) {
                    cb = static_cast<int>(cl >> kClosureSizeBits) - 1;
                    cn = static_cast<int>(cl & kClosureSizeMask) + 1;
                } else {
                    first = lo.w > lo.z;
                    xb = lo.z + 1;
                    xd = max(lo.w - lo.z - 1, 0);
                }
            }
        }
    }
    // closure lists, spread over the wave, kChunks chunks of paths at a time
    {
        const int incl = wave_incl_scan(cn);
        const int pre = incl - cn;
        const int rel = cb - pre;   // entry of a path: rel of its item + the path's place
        const int tot = __builtin_amdgcn_readlane(incl, kWave - 1);
        for (int k0 = 0; k0 < tot; k0 += kWave * kChunks) {
            int o[kChunks], e[kChunks];
            float oc[kChunks];
            bool live[kChunks];
#pragma unroll
            for (int r = 0; r < kChunks; r++) o[r] = owner_scan(pre, cn, k0 + r * kWave);
#pragma unroll
            for (int r = 0; r < kChunks; r++) {
                const int at = k0 + r * kWave + lane;
                live[r] = at < tot;
                e[r] = __shfl(rel, o[r], kWave) + at;
                oc[r] = __shfl(cst, o[r], kWave);
            }
            offer_paths<M, kChunks>(p, t, sh, c, wq, live, e, oc, bnd);
        }
    }
    if (__ballot(first)) {
        // the first epsilon arc, from the state record (the closure word of
        // its destination is not at hand there)
        const float cnd = cst + __int_as_float(x0.y);
        const uint32_t key = okey(cnd);
        offer1<M>(p, t, sh, c, wq, first && key <= bnd, static_cast<uint32_t>(x0.x) & kDstMask, x0.x < 0,
                            0u, cnd, key);
    }
    // the other epsilon arcs, spread over the wave
    const int incl = wave_incl_scan(xd);
    const int pre = incl - xd;
    const int tot = __builtin_amdgcn_readlane(incl, kWave - 1);
    for (int k0 = 0; k0 < tot; k0 += kWave) {
        const int kk = k0 + lane;
        const int o = owner_scan(pre, xd, k0);
        const int ob = __shfl(xb, o, kWave);
        const int op = __shfl(pre, o, kWave);
        const float oc = __shfl(cst, o, kWave);
        bool act = false, d_eps = false;
        uint32_t d = 0, key = kEmptyKey, cw = 0u;
        float cnd = 0.0f;
        if (kk < tot) {
            const int4 r = p.g.xarc[ob + (kk - op)];
            d = static_cast<uint32_t>(r.x) & kDstMask;
            d_eps = r.x < 0;
            cw = static_cast<uint32_t>(r.w);
            cnd = oc + __int_as_float(r.y);
            key = okey(cnd);
            act = key <= bnd;
        }
        offer1<M>(p, t, sh, c, wq, act, d, d_eps, cw, cnd, key);
    }
}

// Relax the wave's queue until it is empty (items pushed meanwhile included).
template <int M>
__device__ __forceinline__ void drain(const Params &p, const Tab<M> &t, Sh &sh, Cnt &c, WaveQ &wq)
{
    const int lane = lane_id();
    while (wq.n > 0) {
        if (__builtin_amdgcn_readfirstlane(c.overflow)) {   // the frame is redone anyway
            wq.n = 0;
            break;
        }
        const int take = min(wq.n, kWave);
        const int base = wq.n - take;
        // items were stored by other lanes of the wave
        wave_lds_handover();
        const uint2 it = lane < take ? wq.q[base + lane] : make_uint2(0u, 0u);
        const uint32_t icl = lane < take ? wq.ql[base + lane] : 0u;
        wq.n = base;
        relax<M>(p, t, sh, c, wq, lane < take, it, icl);
    }
}

// The token set the last frame made (the same in every thread).
struct Set {
    int n, a;        // tokens, emitting out-arcs
    int at, end;     // its survivors, relative to the utterance's region
};

// One frame: produces S_k (set, on success) from S_{k-1} (or from the start
// state when k = 0).  row_k / row_next: original frame of decoded frame k and
// of the next one.  Returns 0, kOverflow (the table filled up; nothing of S_k
// was written) or a negative WFST error.  Every return is taken by the whole
// workgroup.
template <int M>
__device__ __forceinline__ int frame(const Params &p, Lds &lds, const Tab<M> &t, float2 *gcb, const float *ll, int Tp, int row_k,
                                     int row_next, uint2 *spill, int gcap, int k, Set &set, int &n_ins)
{
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    Sh &sh = lds.sh;
    Prof &pf = lds.pf;
    const UttLayout &ly = lds.ly;
    Cnt &c = sh.c[k & 1];
    WaveQ wq;
    wq.q = lds.wq + wid * kQueue;
    wq.ql = lds.wql + wid * kQueue;
    wq.qcap = min(kQueue, p.gen_lds);
    wq.n = 0;
    wq.spill = spill;
    wq.spill_n = &c.spill_n[0];
    wq.scap = gcap;

    phase_mark(p, pf, 5);
    // ---- 1. expansion ----
    sub_open(p, pf);
    if (k == 0) {
        if (wid == 0) {
            const int s = p.g.start;
            const int4 lo = p.g.srec[s];
            offer1<M>(p, t, sh, c, wq, lane == 0, static_cast<uint32_t>(s), lo.w > lo.z, 0u, 0.0f,
                                okey(0.0f));
            if (lane == 0) c.best = okey(0.0f);
        }
    } else {
        const float *grow = ll + static_cast<int64_t>(row_k) * p.L;
        const int64_t at = ly.sv0 + set.at;
        SetView v{nullptr, p.sv_epre + at, p.sv_state + at, p.sv_key + at, chunk_cs<M>(lds), chunk_am<M>(lds), set.n, set.a};
        if constexpr (M == kSmall) {
            v.cb = lds.s.cb;
            v.epre = lds.s.epre;
            expand<M, true>(p, t, sh, c, v, lds.s.row, grow, wq);
        } else if constexpr (M == kBig) {
            v.cb = gcb;
            expand<M, true>(p, t, sh, c, v, lds.s.row, grow, wq);
        } else if (set.n <= kDevSet) {
            v.cb = lds.d.cb;
            expand<M, true>(p, t, sh, c, v, lds.d.row, grow, wq);
        } else {
            expand<M, false>(p, t, sh, c, v, lds.d.row, grow, wq);
        }
    }
    sub_close(p, pf, 4);
    // ---- 2. epsilon closure: each wave its own queue, then spill rounds ----
    drain<M>(p, t, sh, c, wq);
    frame_barrier<M>();
    phase_mark(p, pf, 0);
    // every wave has left frame k - 1: its counters are cleared for frame k + 1
    if (tid == kT - 2 * kWave) sh.c[(k + 1) & 1] = empty_cnt();
    // the next frame's log-likelihood row into LDS, where this frame's is no
    // longer read; the compaction's barrier waits for it
    if (M != kBig && p.L <= kRowMax && k < Tp) {
        const float *nrow = ll + static_cast<int64_t>(row_next) * p.L;
        for (int i0 = wid * kWave; i0 < p.L; i0 += kT)
            fetch_lds(nrow + min(i0 + lane, p.L - 1), lds.s.row + i0);
    }
    if (c.spill_n[0] && !c.overflow && !sh.status) {
        // spilled items are read by other waves
        block_sync_vm();
        int sp = 0;
        while (true) {
            const int total = min(c.spill_n[sp], gcap);
            if (total == 0 || c.overflow || sh.status) break;
            const uint2 *list = spill + static_cast<int64_t>(sp) * gcap;
            if (tid == 0) c.spill_n[sp ^ 1] = 0;
            __syncthreads();
            wq.spill = spill + static_cast<int64_t>(sp ^ 1) * gcap;
            wq.spill_n = &c.spill_n[sp ^ 1];
            for (int c0 = wid * kWave; c0 < total; c0 += kT) {
                const int i = c0 + lane;
                uint2 it = make_uint2(0u, 0u);
                if (i < total) {
                    const unsigned long long w = ldg(reinterpret_cast<const unsigned long long *>(list + i));
                    it = make_uint2(static_cast<uint32_t>(w), static_cast<uint32_t>(w >> 32));
                }
                relax<M>(p, t, sh, c, wq, i < total, it, 0u);
                drain<M>(p, t, sh, c, wq);
            }
            block_sync_vm();
            sp ^= 1;
        }
    }
    phase_mark(p, pf, 1);
    if (c.overflow) {
        phase_fold(p, pf, false);   // the frame is redone on a larger table
        return kOverflow;
    }
    if (sh.status) return sh.status;

    // ---- 3. pruning ----
    const int n = __builtin_amdgcn_readfirstlane(c.nslots);
    n_ins = n;
    const uint32_t kb = c.best;
    const uint32_t lim = beam_limit(kb, p.beam);
    uint32_t cut = lim;
    if (p.max_active > 0 && n > p.max_active && kb <= lim) {
        uint32_t *hist = reinterpret_cast<uint32_t *>(lds.wq);
        int shf = first_shift(kb, lim);
        for (int i = tid; i < kHistBins; i += kT) hist[i] = 0u;
        __syncthreads();
        int cnt = 0;
        for (int i = tid; i < n; i += kT) {
            const uint32_t key = tld<M>(t.vals + t.slots[i]);
            if (key <= lim) {
                cnt++;
                atomicAdd(&hist[(key - kb) >> shf], 1u);
            }
        }
        if (cnt) atomicAdd(&c.cnt, cnt);
        __syncthreads();
        if (c.cnt > p.max_active) {
            int rank = p.max_active;
            select_bin(hist, kHistBins, rank, sh);
            uint32_t prefix = static_cast<uint32_t>(sh.bin) << shf;
            rank -= sh.before;
            while (shf > 0) {
                const int nsh = shf > kHistBits ? shf - kHistBits : 0;
                const int nb = 1 << (shf - nsh);
                __syncthreads();
                for (int i = tid; i < nb; i += kT) hist[i] = 0u;
                __syncthreads();
                for (int i = tid; i < n; i += kT) {
                    const uint32_t key = tld<M>(t.vals + t.slots[i]);
                    if (key > lim) continue;
                    const uint32_t off = key - kb;
                    if ((off >> shf) == (prefix >> shf)) atomicAdd(&hist[(off >> nsh) & (nb - 1)], 1u);
                }
                __syncthreads();
                select_bin(hist, nb, rank, sh);
                prefix |= static_cast<uint32_t>(sh.bin) << nsh;
                rank -= sh.before;
                shf = nsh;
            }
            const uint32_t theta = kb + prefix;
            cut = theta < lim ? theta : lim;
        }
        __syncthreads();
    }

    phase_mark(p, pf, 2);

    // ---- 4. compaction into S_k ----
    // Each wave takes chunks of the slot list, clears their slots, loads the
    // survivors' state records together and places its survivors with one
    // 64-bit LDS add of (emitting degrees << 32 | count): the returned value
    // gives their positions and the prefix of emitting degrees before them
    // at once.  The order of a token set is internal (sets are reported
    // sorted by state), so no block-wide scan is needed.
    const int set0 = set.end;
    int xacc = 0, zacc = 0;   // this lane's survivors: epsilon degrees, how many have no emitting arc
    for (int i0 = wid * kWave; i0 < n; i0 += kT) {
        const int i = i0 + lane;
        const bool in = i < n;
        const uint32_t sl = static_cast<uint32_t>(t.slots[min(i, n - 1)]);
        const uint32_t vv = tld<M>(t.vals + sl);
        const int dd = static_cast<int>(tld<M>(t.keys + sl));
        const bool kp = in && vv <= cut;
        const int4 lo = p.g.srec[in ? dd : 0];
        if (in) {
            t.keys[sl] = kEmptyKey;
            t.vals[sl] = kEmptyKey;
        }
        // (lo is used on every path: a load left pending into the next round
        // would make that round wait before writing its registers)
        const uint64_t km = __ballot(kp);
        const int tc = __popcll(km);
        const int deg = kp ? lo.y - (dd + 2) : 0;   // (at least one record)
        xacc += kp ? lo.w - lo.z : 0;
        zacc += kp && lo.x == 0;
        const int id = wave_incl_scan(deg);
        const int td = __builtin_amdgcn_readlane(id, kWave - 1);
        unsigned long long base = 0;
        if (lane == 0 && tc)
            base = atomicAdd(&c.alloc, (static_cast<unsigned long long>(td) << 32) | static_cast<uint32_t>(tc));
        const int pos = __builtin_amdgcn_readlane(static_cast<int>(base), 0) + rank_in(km);
        const int apos = __builtin_amdgcn_readlane(static_cast<int>(base >> 32), 0) + id - deg;
        if (!kp) continue;
        if (M == kSmall && pos < kSetCache) {
            // to the survivor arrays after the barrier below
            lds.s.cb[pos] = make_float2(okey_val(vv), __int_as_float(dd + 2 - apos));
            lds.s.epre[pos] = apos;
        } else if (static_cast<int64_t>(set0) + pos < ly.svcap) {
            const int64_t o = ly.sv0 + set0 + pos;
            p.sv_state[o] = dd;
            p.sv_key[o] = vv;
            p.sv_epre[o] = apos;
            if (M == kBig && pos < kBigFill) gcb[pos] = make_float2(okey_val(vv), __int_as_float(dd + 2 - apos));
        }
        if (M == kDev && pos < kDevSet) lds.d.cb[pos] = make_float2(okey_val(vv), __int_as_float(dd + 2 - apos));
        mark_begin(chunk_cs<M>(lds), chunk_am<M>(lds), kChunksMax<M>, apos, deg, pos);
    }
    {
        const int tx = wave_incl_scan(xacc), tz = wave_incl_scan(zacc);
        if (lane == kWave - 1 && (tx | tz))
            atomicAdd(&c.xsum, (static_cast<unsigned long long>(tz) << 32) | static_cast<uint32_t>(tx));
    }
    // the next row has arrived (and with the slot list or the table in device
    // memory the survivors' stores and the cleared slots)
    fetch_wait();
    frame_barrier<M>();
    const unsigned long long alloc = c.alloc;
    const int ns = __builtin_amdgcn_readfirstlane(static_cast<int>(alloc));
    const int a_kept = __builtin_amdgcn_readfirstlane(static_cast<int>(alloc >> 32));
    // The survivors placed in the LDS copy go to the survivor arrays now, in
    // one batch of stores that overlaps the next frame's start (a state's id
    // is its first emitting unit minus 2).  Stores inside the loop above
    // would make each of its rounds wait for them.
    if (static_cast<int64_t>(set0) + ns > ly.svcap) return WFST_ECAPACITY;
    if constexpr (M == kSmall) {
        for (int i = tid; i < min(ns, kSetCache); i += kT) {
            const int64_t o = ly.sv0 + set0 + i;
            const float2 x = lds.s.cb[i];
            const int32_t ep = lds.s.epre[i];
            p.sv_state[o] = __float_as_int(x.y) + ep - 2;
            p.sv_key[o] = okey(x.x);
            p.sv_epre[o] = ep;
        }
    }
    phase_mark(p, pf, 3);
    phase_fold(p, pf, true);
    if (ns == 0) return WFST_ENOPATH;
    // Token set k, its cutoff and the lattice record regions of set k: one
    // record per emitting arc of S_k (into S_k+1) at most, one per epsilon
    // arc of S_k at most; a dead end's placeholder arc gives no record and
    // reserves none, so the record pass gets the set's arcs with the
    // placeholders apart.  (A region that would overflow is reported through
    // sh.status: the next frame sees it after its first barrier, and the set
    // is not published.)
    if (tid == kT - kWave) {
        Run &run = lds.run;
        const int64_t a_rec = k < Tp ? a_kept - static_cast<int>(c.xsum >> 32) : 0;
        const int x_kept = static_cast<int>(c.xsum);
        // (with the incremental lattice pass the regions only bound the ring use
        // per set; the pass checks its own capacities)
        if (p.lattice && !p.stream_k && (run.le + a_rec > ly.lecap || run.lx + x_kept > ly.lxcap)) {
            sh.status = WFST_ECAPACITY;
        } else {
            run.le += a_rec;
            run.lx += x_kept;
            run.eps += x_kept;
            p.set_arcs[ly.fo0 + k] = a_kept;
            p.sv_off[ly.fo0 + k + 1] = set0 + ns;
            p.cut_arr[ly.fo0 + k] = cut;
            p.rle_off[ly.fo0 + k + 1] = run.le;
            p.rlx_off[ly.fo0 + k + 1] = run.lx;
        }
    }
    set.n = ns;
    set.a = a_kept;
    set.at = set0;
    set.end = set0 + ns;
    return 0;
}

// ---------------------------------------------------------------------------
// Record workgroups beside the search.  A launch may carry rec_wg workgroups
// after its U search workgroups (they are dispatched after them).  They
// derive the back-pointers and raw lattice records of the launch's token
// sets (record_one, the record kernel's work) while the search still runs,
// so that the record pass of the batch's longest utterances ends with their
// search instead of after it.  Items (token set k, utterance u) are taken in
// frame order from a device counter; item (k, u) needs sets k - 1 and k,
// i.e. a published count prog[u] > k (the search publishes every pub_k sets
// and at its end; -1 when it failed).  Thread 0 polls the count with relaxed
// loads; wave 0 then reads every utterance's count into seen[] and takes one
// acquire fence, which makes visible everything those counts cover.  The
// fence invalidates the caches that the searches of the chiplet share, so a
// workgroup takes one only when an item needs a set beyond seen[].
// ---------------------------------------------------------------------------
constexpr long long kRecPolls = 1LL << 22;  // polls of one count (several seconds) before giving up

struct RecLds {
    RSh rsh;
    int item;
    int prog;
    int seen[kRecMaxUtts];
    RecMid l;
};

__device__ __forceinline__ void record_role(const Params &p, RecLds &r)
{
    const int U = p.U;
    const int items = (p.rec_tmax + 1) * U;
    const int tid = threadIdx.x;
    for (int i = tid; i < U; i += blockDim.x) r.seen[i] = 0;
    while (true) {
        if (tid == 0) r.item = atomicAdd(p.rec_next, 1);
        __syncthreads();
        const int i = r.item;
        if (i >= items) break;
        const int k = i / U;
        const int u = i - k * U;
        UttState &st = p.st[u];
        // every thread has read the item before thread 0 takes the next
        if (k > st.Tp || r.seen[u] < 0) {
            __syncthreads();
            continue;
        }
        if (r.seen[u] <= k) {
            if (tid == 0) {
                int v = 0;
                for (long long n = 0;; n++) {
                    v = __hip_atomic_load(p.prog + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (v > k || v < 0) break;
                    // another record workgroup may have given up on it already
                    if (n >= kRecPolls || __hip_atomic_load(&st.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                                              kStatusStreamTimeout) {
                        v = -2;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(32);
                }
                if (v == -2) set_status(st, kStatusStreamTimeout);
                r.prog = v;
            }
            // (seen[] is written only after every thread has read it above)
            __syncthreads();
            if (r.prog > k) {
                if (tid < kWave) {
                    // the counts as they are now; the fence covers them all
                    for (int w = tid; w < U; w += kWave) {
                        const int v = __hip_atomic_load(p.prog + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        r.seen[w] = v < 0 ? -1 : max(r.seen[w], v);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                }
            } else if (tid == 0) {
                // the search failed, or the wait gave up: the utterance's
                // remaining items are skipped
                r.seen[u] = -1;
            }
            __syncthreads();
            if (r.seen[u] <= k) continue;
        }
        const int n = set_size(p, p.lay[u], k);
        if (n <= min(kRFill, p.rec_fill)) record_one(p, u, k, n, r.l, r.rsh);
        else if (tid == 0) atomicOr(&st.big_sets, kSetLarge);   // left to the large-set pass
        __syncthreads();
    }
}

template <bool kRec>
__global__ __launch_bounds__(kT) void search_kernel(Params p)
{
    // All LDS in one struct, the small fields first: they then lie below
    // 64 KB, where an LDS instruction reaches them with an immediate offset
    // instead of an address held in a register.
    union All {
        Lds s;
        RecLds r;
    };
    static_assert(sizeof(RecLds) <= sizeof(Lds), "the record workgroups fit the search's LDS");
    __shared__ All all;
    Lds &lds = all.s;
    if constexpr (kRec) {
        if (static_cast<int>(blockIdx.x) >= p.U) {
            record_role(p, all.r);
            return;
        }
    }
    Sh &sh = lds.sh;
    Prof &pf = lds.pf;

    const int u = blockIdx.x;
    const int tid = threadIdx.x;
    UttState &st = p.st[u];
    if (st.status != 0) {
        if (p.pub_k && tid == 0) publish_release(p.prog + u, -1);
        return;
    }
    // the layout is copied into LDS: a reference into device memory would be
    // reloaded after every barrier, and a copy in registers would hold a
    // dozen of them for the whole kernel
    if (tid == 0) {
        lds.ly = p.lay[u];
        lds.run = Run{};
        sh.status = 0;
        for (int i = 0; i < 2; i++) sh.c[i] = empty_cnt();
        for (int i = 0; i < 7; i++) pf.ph[i] = 0;
        for (int i = 0; i < 4; i++) pf.cur[i] = 0;
        pf.t_last = wall_clock64();
        pf.t_sub = 0;
    }
    for (int i = tid; i < kSlots; i += kT) {
        lds.s.keys[i] = kEmptyKey;
        lds.s.vals[i] = kEmptyKey;
    }
    for (int i = tid; i < kCs; i += kT) lds.am[i] = make_uint2(0u, 0u);
    __syncthreads();
    const UttLayout &ly = lds.ly;
    const int Tp = st.Tp;
    const float *ll = st.ll;

    const Tab<kSmall> lt{lds.s.keys, lds.s.vals, lds.s.slots, kSlots, min(kFill, p.lds_fill), 32 - kSlotBits,
                         p.hash_mul};
    const int64_t gbase = static_cast<int64_t>(u) * p.capG;
    // (the device-memory table is never smaller than kBigFill entries; while
    // the big table is in use its keys hold the set's costs and positions)
    float2 *gcb = reinterpret_cast<float2 *>(p.gkeys + gbase);
    const Tab<kBig> bt{lds.b.keys, lds.b.vals, p.gslots + gbase, kBigSlots, min(kBigFill, p.lds_fill), 32 - kBigBits,
                       p.hash_mul};
    const Tab<kDev> gt{p.gkeys + gbase, p.gvals + gbase, p.gslots + gbase, static_cast<uint32_t>(p.capG),
                       static_cast<int>(p.capG / 4 * 3), 32 - (31 - __clz(static_cast<int>(p.capG))), p.hash_mul};
    const int gcap = static_cast<int>(p.capO);
    uint2 *spill = p.gspill + static_cast<int64_t>(u) * 2 * p.capO;

    Set set{0, 0, 0, 0};
    int gframes = 0;       // frames on the device-memory table (thread 0's count)
    int mode = kSmall;     // the table the LDS is set up for
    bool dev_clean = false;   // the device-memory table holds no token
    int want = kSmall;     // the table of the next frame
    int rc = 0;
    int row_k = 0, row_next = Tp > 0 ? p.kept[ly.kept0] : 0;   // original frames of decoded frame k and the next
    for (int k = 0; k <= Tp; k++) {
        const int row_after = k + 1 < Tp ? p.kept[ly.kept0 + k + 1] : 0;
        int n_ins = 0;
        for (;;) {
            if (want != mode) {
                // the other table: the set is read where that one expects it
                // (its stores, and fetches into the LDS, complete first)
                fetch_wait();
                block_sync_vm();
                if (want == kDev) {
                    if (!dev_clean) {
                        for (int64_t i = tid; i < p.capG; i += kT) {
                            gt.keys[i] = kEmptyKey;
                            gt.vals[i] = kEmptyKey;
                        }
                        dev_clean = true;
                    }
                } else {
                    uint32_t *keys = want == kBig ? lds.b.keys : lds.s.keys;   // (values follow keys)
                    const int words = 2 * (want == kBig ? kBigSlots : kSlots);
                    for (int i = tid; i < words; i += kT) keys[i] = kEmptyKey;
                    if (want == kBig) dev_clean = false;
                }
                uint2 *am = want == kDev ? lds.d.am : lds.am;
                uint16_t *cs = want == kDev ? lds.d.cs : lds.cs;
                const int nch = want == kDev ? kDevCs : kCs;
                for (int i = tid; i < nch; i += kT) am[i] = make_uint2(0u, 0u);
                __syncthreads();
                // the set where this table's frames read it, its chunks, and the row
                for (int i = tid; i < set.n; i += kT) {
                    const int64_t o = ly.sv0 + set.at + i;
                    const int32_t ep = p.sv_epre[o];
                    const float2 x = make_float2(okey_val(p.sv_key[o]), __int_as_float(p.sv_state[o] + 2 - ep));
                    if (want == kBig) {
                        gcb[i] = x;
                    } else if (want == kSmall) {
                        lds.s.cb[i] = x;
                        lds.s.epre[i] = ep;
                    } else if (i < kDevSet) {
                        lds.d.cb[i] = x;
                    }
                    mark_begin(cs, am, nch, ep, (i + 1 < set.n ? p.sv_epre[o + 1] : set.a) - ep, i);
                }
                if (want != kBig && k > 0 && p.L <= kRowMax)
                    for (int i = tid; i < p.L; i += kT)
                        lds.s.row[i] = ldg(ll + static_cast<int64_t>(row_k) * p.L + i);
                block_sync_vm();
                mode = want;
            }
            if (want == kSmall) rc = frame<kSmall>(p, lds, lt, gcb, ll, Tp, row_k, row_next, spill, gcap, k, set, n_ins);
            else if (want == kBig) rc = frame<kBig>(p, lds, bt, gcb, ll, Tp, row_k, row_next, spill, gcap, k, set, n_ins);
            else rc = frame<kDev>(p, lds, gt, gcb, ll, Tp, row_k, row_next, spill, gcap, k, set, n_ins);
            if (rc != kOverflow) break;
            if (want == kDev) {
                rc = WFST_ECAPACITY;
                break;
            }
            // (the abandoned attempt left states in the LDS table, which is
            // cleared before it is used again) the frame's counters start over
            __syncthreads();
            if (tid == 0) sh.c[k & 1] = empty_cnt();
            want++;
        }
        if (want == kDev) gframes++;
        if (rc != 0) break;
        // The next frame's table.  A set beyond the small table's LDS copy
        // needs the big one; after a frame that needed a larger table, the
        // next frames stay there while their tables are close to the smaller
        // one's limit: a frame started there would most likely be abandoned
        // half-way.
        if (want == kDev && n_ins > bt.fill - bt.fill / 8) want = kDev;
        else if (set.n > kSetCache || (want != kSmall && n_ins > lt.fill - lt.fill / 8)) want = kBig;
        else want = kSmall;
        row_k = row_next;
        row_next = row_after;
        // publish every pub_k finished token sets to the record workgroups
        // or the incremental lattice pass: every wave's stores of the sets
        // complete in L2 first (the last barrier of a frame orders LDS only),
        // then one release store of the count (which writes the cache back
        // for readers possibly on another chiplet)
        if (p.pub_k && (k + 1) % p.pub_k == 0 && k < Tp) {
            block_sync_vm();
            if (tid == 0 && sh.status == 0) publish_release(p.prog + u, k + 1);
        }
    }
    // (the workgroup's LDS is not given back while a fetch into it is under way)
    fetch_wait();
    block_sync_vm();
    if (tid == 0) {
        if (rc == 0) rc = sh.status;
        st.n_tok = set.end;
        st.n_last = set.n;
        st.arcs_expanded = lds.run.le;
        st.eps_arcs = lds.run.eps;
        st.gframes = gframes;
        for (int i = 0; i < 7; i++) st.phase_ticks[i] = pf.ph[i];
        if (rc != 0) st.status = rc;
        if (p.pub_k) {
            vm_wait();
            publish_release(p.prog + u, rc == 0 ? Tp + 1 : -1);
        }
    }
}

}  // namespace

}  // namespace wfd
