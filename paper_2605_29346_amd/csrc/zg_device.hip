// HIP kernels (gfx950, wave64) and the plan / step entry points of libzg.
//
// One step = H+2 launches: the hop kernel's launches 0..H-1, the closing launch and {aggregate + relabel of the last hop +
// finish} (H+3 when X is written by a gather launch of its own; a small step's hops are one workgroup's work: 2, or 3).  Launch l of
// the hop kernel samples hop l and, for l > 0, first ranks the vertices hop l-1 discovered - they are rows of block l
// themselves, so ranking and sampling share their chained scans; launch 0 also ingests the seeds, launch l >= 2 relabels the
// edges of hop l-2 and the closing launch ranks only (workgroups of a launch are split by role).
// Every kernel boundary costs about as much as the small kernels themselves at mini-batch sizes, and kernels of
// different streams do not hide it from each other, so the step is cut into as few launches as its global
// dependencies allow: "all of hop l-1 sampled" before its vertices can be ranked, and "all vertices ranked" before
// the features move.
// Every kernel is launched with a grid fixed by the plan's capacity envelope, reads the true sizes
// from the device-resident metadata buffer and lets surplus workgroups return at once (paper
// sections 4.1-4.3).  The launches are the same for every step but for the seeds pointer and the key, which its first one
// takes as arguments; with a twin behind it the step is one hipGraph (section 4.4) and takes them through a mailbox in pinned
// host memory (see issue_step).
// A plan may carry a worst-case twin (the paper's "cached safe graph", section 4.3) that replays a mini-batch
// whose sizes overflowed the envelope, on the host's request or - its kernels appended to the step's graph
// behind a device-side gate - by itself.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>

#include "zg_floyd.h"
#include "zg_internal.h"

namespace zg {

// =================================================================================================
// device helpers
// =================================================================================================
// four floats moved as one access, at any float's address: the memory system takes 16 bytes at a 4-byte boundary in one
// instruction, so rows of any width >= 4 and any stride go this way
typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));

constexpr uint64_t kStAggregate = 1ull << 62; // status word of a ticket: its total published ...
constexpr uint64_t kStPrefix = 2ull << 62;    // ... or its inclusive prefix
constexpr uint32_t kPatience = 256;           // polls, about a microsecond each, before a workgroup does what it waits for itself
constexpr uint32_t kSpinLimit = 1u << 22;     // ... where its predecessors are known to run: before it gives up with ZG_FLAG_INTERNAL

// value of the lane a DPP control names, 0 where there is none
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}

// inclusive sum over the wavefront's lanes, all of them active: six register moves (a shuffle through LDS per step costs the
// latency-bound launches about 0.3 us per scan)
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xF>(v); // row_shr:1, 2, 4, 8: within rows of 16 lanes
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    v += dpp_or_zero<0x142, 0xA>(v); // row_bcast:15: last lane of rows 0 and 2 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v); // row_bcast:31: lane 31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane); }
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return lane_value(wave_incl_scan(v), 63u); }

__device__ __forceinline__ void st_store(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t st_load(uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Single-pass chained scan across workgroups, in the order of their tickets (a ticket: one workgroup's share of a launch, by
// workgroup index).  Ticket t publishes its total, and later looks back over the predecessors' status words until it meets a
// published inclusive prefix.  A status word carries state and value together, so one relaxed 64-bit access is enough.  One
// wavefront looks back, 64 predecessors per round.  (Measured and not kept: sharing a look-back among eight wavefronts -
// the wait is for the predecessors to publish, not for the rounds; a second level of one word per 32 tickets that each
// ticket adds to and every later ticket polls - the polls of one line queue up behind each other, launches of 400
// tickets took twice as long.)
// Whether a predecessor is running while a workgroup waits for it depends on what a ticket is (see k_hop).  Drawn from a counter, in
// the order in which workgroups start: all of them are, and the lowest unfinished one never waits.  The workgroup's index: kernels of
// other streams may hold the compute units it needs, and wait in turn for workgroups that this kernel keeps out.  So a wait ends after `patience` polls:
// `missing(t)` then works out ticket t's total from what the launch found - which t changes only after its totals are published
// (publish_done), so that what was read stands if they still are not.  It does so for the nearest ticket, then looks at all of them again,
// and asks for none beyond the nearest prefix.  (All that were missing at the first look, one after another: steps with no patience
// at all took 454 us where patient ones take 113, now 120; 370 where 96, now 102.)  No wait depends on another workgroup's progress, and no wait changes
// the result.  Where the marks are changed before the totals are published, and tickets always drawn, the wait is bounded all the same
// (kSpinLimit): when it runs out the step is flagged invalid (sticky and per-step word) and what is there is used.
// Values are taken modulo 2^32: more than that is only reached beyond a cap, by dropped rows.
__device__ __forceinline__ void chain_publish(uint64_t *status, uint32_t t, uint32_t total)
{
    st_store(&status[t], (t == 0u ? kStPrefix : kStAggregate) | total);
}

// the publishing wavefront's stores have been performed; behind a barrier the workgroup may change what its totals were taken from (the wavefront
// that publishes is one that looks back: chain_prefix ends with this)
__device__ __forceinline__ void publish_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// all 64 lanes of one wavefront: the sum of the totals of tickets 0 .. t-1, after this ticket's own was published.  A look goes
// back WINDOWS windows of 64 tickets, all their status words on the way at once.  Four in launch 0 and for the closing launch's tiles of words, whose tickets publish at
// about the same time and find no prefix nearby: with a window per look, a microsecond each, the last of 235 tickets had its sum 6 us
// after the last total was published, now 2 us.  One where what is waited for is other tickets' loads (a launch of 2 M edges 47.2 us, with
// four 49.4).
template <int WINDOWS, class Missing>
__device__ __forceinline__ uint32_t chain_prefix(uint64_t *status, uint32_t t, uint32_t total, Drmb *d, int lane, uint32_t patience, const Missing &missing)
{
    uint32_t excl = 0, polls = 0;
    if (t == 0u) {
        publish_done();
        return 0u;
    }
    uint32_t worked_out = 0;         // this lane's ticket's total in the first window, ...
    unsigned long long known = 0ull; // ... where it had to be
    for (int64_t base = (int64_t)t - 1;;) {
        // window w: the status words base - 64 w, .. of 64 tickets (indices below zero count as an inclusive prefix of zero)
        uint64_t st[WINDOWS];
#pragma unroll
        for (int w = 0; w < WINDOWS; ++w) {
            const int64_t idx = base - 64 * w - lane;
            st[w] = idx >= 0 ? st_load(&status[idx]) : kStPrefix;
        }
        if ((st[0] >> 62) == 0 && ((known >> lane) & 1ull)) st[0] = kStAggregate | worked_out;
        unsigned long long none = 0ull, pm = 0ull; // of the last window looked at: tickets whose total is not there, those whose prefix is
#pragma unroll
        for (int w = 0; w < WINDOWS; ++w) {
            if (none || pm) break;
            pm = __ballot((st[w] >> 62) == 2);
            none = __ballot((st[w] >> 62) == 0) & (pm ? (pm & (0ull - pm)) - 1ull : ~0ull); // (none beyond the nearest prefix)
            if (none) break;
            excl += wave_sum(lane <= (pm ? __ffsll((long long)pm) - 1 : 63) ? (uint32_t)st[w] : 0u);
            base -= 64;
            known = 0ull;
        }
        if (!none) {
            if (pm) break;
            continue;
        }
        if (++polls > patience) {
            if (patience == kSpinLimit) { // drawn tickets: the step's outputs are invalid, both the sticky and the per-step word say so
                if (lane == 0) {
                    atomicOr(&d->flags, ZG_FLAG_INTERNAL);
                    atomicOr(&d->step_flags, ZG_FLAG_INTERNAL);
                }
                break;
            }
            // the nearest one; then another look at all of them: the others, or a prefix, may be there by now
            const int l = __ffsll((long long)none) - 1;
            const uint32_t v = missing((uint32_t)(base - l));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // read before that look
            if (lane == l) worked_out = v;
            known |= 1ull << l;
            continue;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    publish_done(); // (with the looks behind it nothing is left to wait for)
    if (lane == 0) st_store(&status[t], kStPrefix | (uint32_t)(excl + total));
    return excl;
}

// a * b in one instruction (the compiler makes two products of it, low half and high half)
__device__ __forceinline__ uint64_t product(uint32_t a, uint32_t b)
{
    uint64_t p;
    asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(p) : "v"(a), "s"(b) : "vcc");
    return p;
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

// Philox4x32-10 (Salmon et al., SC'11) for counter (node, slot, hop, 0) and the 64-bit step key;
// returns the first two output words as one 64-bit draw.  A sampling pass computes this more than anything else: 36
// products and as many pairs of xors took 114 ns per wavefront with 8 of them on a SIMD, 20 whole products and three-way xors
// take 73 ns.
__device__ __forceinline__ uint64_t philox_draw(uint32_t key_lo, uint32_t key_hi, uint32_t hop, uint32_t node, uint32_t slot)
{
    uint32_t c0 = node, c1 = slot, c2 = hop, c3 = 0u;
    uint32_t k0 = key_lo, k1 = key_hi;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = product(c0, 0xD2511F53u);
        const uint64_t p1 = r == 0 ? (uint64_t)0xCD9E8D57u * c2 : product(c2, 0xCD9E8D57u); // (the first one is the hop's: a scalar)
        c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        c1 = (uint32_t)p1;
        c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return (uint64_t)c0 | ((uint64_t)c1 << 32);
}

// floor(x * b / 2^64) for a 32-bit b: two 32 x 32 products instead of a 64 x 64 one
__device__ __forceinline__ uint32_t scale_draw(uint64_t x, uint32_t b)
{
    return (uint32_t)(((x >> 32) * b + (((x & 0xFFFFFFFFull) * b) >> 32)) >> 32);
}

// The wavefront as the interface of floyd_position (zg_floyd.h): F consecutive lanes from gbase on hold the slots of this lane's frontier
// vertex.  A flag is looked up in the wavefront's mask of them.
struct WaveGroup {
    uint32_t gbase;
    __device__ __forceinline__ uint32_t up(uint32_t x) const { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, true); } // wave_shr:1
    __device__ __forceinline__ bool flag_of(uint32_t j, bool mine) const { return (__ballot(mine) >> (gbase + j)) & 1ull; }
    __device__ __forceinline__ bool any(bool b) const { return __any(b) != 0; }
};

// =================================================================================================
// kernels
// =================================================================================================
// Per-step inputs travel through a ring in pinned host memory that the device reads directly: the captured
// graph's arguments are frozen, and a step must be exactly one graph launch.  The host writes slot
// (steps issued % kMailboxSlots) before it launches the graph; the ingest kernel of step number e (the
// device-side step counter) reads slot e % kMailboxSlots; the last kernel of a step publishes e + 1 in
// `completed`, and how many of those steps the host has enqueued itself - the others are replays of a caller's recording - in `answered`,
// which it checks (no device synchronisation) before it reuses a slot.
struct Mailbox {
    uint32_t completed;
    uint32_t issued; // steps the host has handed over so far (their slots are filled)
    uint32_t answered;
    uint32_t pad;
    uint32_t status[kMailboxSlots]; // ZG_FLAG_* bits raised by the step that used the slot
    struct {
        unsigned long long seeds; // device address of the step's seed ids
        unsigned long long key;   // step key
    } slot[kMailboxSlots];
};

// Device-side conditional of the overflow-safe fallback (paper section 4.3): the worst-case twin's kernels sit
// behind the plan's own in the same captured graph and every one of their workgroups returns at once unless
// the plan's step raised a hop-overflow bit - a fixed launch skeleton whose surplus work exits early, like
// the over-provisioned grids of section 4.2.  `gate` is the plan's metadata buffer (null: always run).
constexpr uint32_t kHopOverflowMask = 0xFFFFu;
__device__ __forceinline__ bool gate_closed(const Drmb *gate)
{
    return gate != nullptr && (gate->last_flags & kHopOverflowMask) == 0u;
}

// The step's inputs as arguments of its first launch (seeds == null: a captured graph's arguments are frozen, they come through the mailbox)
struct StepInputs {
    const int32_t *seeds;
    unsigned long long key;
};

struct IngestArgs {
    StepInputs in;
    Drmb *drmb;
    const Drmb *gate;       // gated twin: the step's inputs are those of the gate owner's step that has just finished
    const Mailbox *mailbox; // the mailbox the inputs are read from (the gate owner's when gated)
    int32_t *S;
    int32_t *local_id;
    uint32_t *seen;
    uint32_t batch;
    uint32_t num_nodes;
    uint32_t blocks; // workgroups given to this role (0: role absent)
};

// The step's (seeds pointer, key).  A read of the pinned-host mailbox costs the device several microseconds, at the head
// of the step's dependency chain; when the host runs ahead of the device - the normal case in a training loop - the
// previous step has already copied this step's slot into the metadata buffer (prefetch_step_inputs) and the read
// stays in device memory.  Otherwise: the mailbox slot of the device-side step counter.
__device__ __forceinline__ bool prefetched_inputs(const Drmb *d, const Drmb *gate, unsigned long long *out)
{
    // (all of it on its way at once: a branch in between would make two round trips of it)
    const uint32_t valid = d->pre_valid, pre_epoch = d->pre_epoch, epoch = d->epoch;
    out[0] = d->pre_seeds;
    out[1] = d->pre_key;
    return !gate && valid && pre_epoch == epoch;
}

__device__ __forceinline__ void mailbox_inputs(const Drmb *d, const Drmb *gate, const Mailbox *mailbox, unsigned long long *out)
{
    const uint32_t slot = (gate ? gate->epoch - 1u : d->epoch) % kMailboxSlots;
    out[0] = __hip_atomic_load(&mailbox->slot[slot].seeds, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    out[1] = __hip_atomic_load(&mailbox->slot[slot].key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One lane of a sampling ticket, where nothing was prefetched (the host waits for every step, or this is the first): ticket 0 reads
// the mailbox and passes the inputs on in device memory.  Reads of host memory queue up: 132 workgroups that each read the
// slot took 20 us.  (The ingest workgroups of the launch, one per 1024 seeds, read it themselves.)  A wait that runs out - ticket 0 need
// not be running yet - reads the mailbox itself.
__device__ __forceinline__ void shared_inputs(Drmb *d, const Drmb *gate, const Mailbox *mailbox, uint32_t ticket, uint32_t patience, unsigned long long *out)
{
    const uint32_t tag = d->epoch + 1u;
    if (ticket != 0u) {
        for (uint32_t polls = 0; polls < patience; ++polls) {
            if (__hip_atomic_load(&d->cur_epoch, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == tag) {
                out[0] = __hip_atomic_load(&d->cur_seeds, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                out[1] = __hip_atomic_load(&d->cur_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    mailbox_inputs(d, gate, mailbox, out);
    if (ticket == 0u) {
        __hip_atomic_store(&d->cur_seeds, out[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&d->cur_key, out[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&d->cur_epoch, tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Step entry ("ingest"): seeds -> D_0 (caller's order), their local ids and "seen" bits; step key and batch size ->
// metadata buffer.  Out-of-range seeds are replaced by -1 (a vertex with no neighbors); a seed whose "seen" bit
// is already set is a duplicate.  Shares its launch with the sampling of hop 0, which reads the seeds itself.
__device__ __forceinline__ void ingest_block(const IngestArgs &a, uint32_t block, unsigned long long *s_in)
{
    const uint32_t gtid = block * blockDim.x + threadIdx.x;
    if (threadIdx.x == 0) {
        if (a.in.seeds) {
            s_in[0] = reinterpret_cast<unsigned long long>(a.in.seeds);
            s_in[1] = a.in.key;
        } else if (!prefetched_inputs(a.drmb, a.gate, s_in)) {
            mailbox_inputs(a.drmb, a.gate, a.mailbox, s_in); // (a workgroup per 1024 seeds)
        }
    }
    __syncthreads();
    const int32_t *seeds = reinterpret_cast<const int32_t *>(s_in[0]);
    if (gtid == 0) {
        Drmb *d = a.drmb;
        d->step = d->epoch;
        d->n[0] = a.batch;
        d->n_exact[0] = a.batch;
        d->key_lo = (uint32_t)(s_in[1] & 0xFFFFFFFFull);
        d->key_hi = (uint32_t)(s_in[1] >> 32);
    }
    if (gtid < a.batch) {
        int32_t v = seeds[gtid];
        if ((uint32_t)v >= a.num_nodes) {
            atomicOr(&a.drmb->flags, ZG_FLAG_SEED_RANGE);
            atomicOr(&a.drmb->step_flags, ZG_FLAG_SEED_RANGE);
            v = -1;
        } else {
            const uint32_t bit = 1u << (v & 31);
            const uint32_t old = atomicOr(&a.seen[(uint32_t)v >> 5], bit);
            if (old & bit) {
                atomicOr(&a.drmb->flags, ZG_FLAG_SEED_DUP);
                atomicOr(&a.drmb->step_flags, ZG_FLAG_SEED_DUP);
            }
            a.local_id[v] = (int32_t)gtid;
        }
        a.S[gtid] = v;
    }
}

// The last hop's new vertices carry, in the top bits of their id-map entry, the tag of the edge whose mark was the last to
// land on the vertex's byte: that edge - and the odd other edge to the vertex with the same tag, which stores the same bytes -
// writes the vertex's row of X.  As many tag bits as the node cap leaves of an int32's 31 (at most 7); with none left every
// edge to a new vertex writes its row.
// In a step whose frontier has `reach_rows` vertices or more, those of them that the last hop reaches again carry a tag too, and their rows are
// written the same way instead of being copied (see gather_unreached_block).
struct MarkTag {
    int32_t shift; // tag = entry >> shift; 0: entries are plain local ids
    uint32_t mask; // tag bits in use
    uint32_t reach_rows;
    __device__ __forceinline__ int32_t entry(uint32_t lid, uint32_t mark) const { return shift ? (int32_t)(lid | ((mark & mask) << shift)) : (int32_t)lid; }
    __device__ __forceinline__ int32_t local_id(int32_t e) const { return shift && e >= 0 ? e & (int32_t)((1u << shift) - 1u) : e; }
    __device__ __forceinline__ bool owns(int32_t e, uint32_t edge) const { return shift == 0 || ((uint32_t)e >> shift) == (edge & mask); }
    __device__ __forceinline__ bool reaches(uint32_t frontier) const { return frontier >= reach_rows; }
};

struct RelabelArgs {
    const Drmb *drmb;
    const Drmb *gate; // consulted by the gather launch (the hop kernel has its own)
    const int32_t *nbr;
    const int32_t *local_id;
    int32_t *col;
    MarkTag tag; // closing launch: how entries carry it, where other workgroups of the launch are adding it
    uint32_t num_nodes;
    int32_t hop;
    uint32_t blocks; // workgroups given to this role (0: role absent)
};

// Hop h, "relabel edges": col[e] = local id of nbr_gid[e] (-1 for a vertex dropped by an overflow).
// Every sampled id is in S_h, so its map entry was written during this step (by the ingest or a ranking tile).
// An entry at or beyond n_{h+1} belongs to a vertex that this hop's cap dropped and a later hop found again - ranked
// by the very launch this role runs in, and on the last hop tagged (MarkTag): the vertex is not in S_h, whichever entry is read.
// Works for any workgroup size; a workgroup covers kRelabelPerBlock edges.
__device__ __forceinline__ void relabel_block(const RelabelArgs &a, uint32_t block)
{
    const uint32_t E = a.drmb->E[a.hop], n = a.drmb->n[a.hop + 1];
    const uint32_t e0 = block * kRelabelPerBlock;
    if (e0 >= E) return;
    const uint32_t e1 = e0 + kRelabelPerBlock < E ? e0 + kRelabelPerBlock : E;
#pragma unroll 4
    for (uint32_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
        const int32_t g = a.nbr[e];
        const int32_t id = a.tag.local_id((uint32_t)g < a.num_nodes ? a.local_id[g] : -1);
        a.col[e] = (uint32_t)id < n ? id : -1;
    }
}

struct RowArgs {
    const float *src;       // gather: feature table; aggregate: input rows
    float *dst;
    const int32_t *S;       // gather: global ids of the rows to copy
    const int32_t *row_ptr; // aggregate
    const int32_t *col;     // aggregate: per edge, the index of its input row (local ids, or - where col_out is set - global ids)
    const uint32_t *n_rows; // device address of the row count
    const uint32_t *n_cols; // aggregate: device address of the block's number of columns: an id at or beyond it is none (where ids come
                            // from the id map: not of this step but a twin's, see mark_tag)
    uint32_t col_limit;     // aggregate whose `col` holds global ids: the number of input rows (num_nodes)
    float *x_dst;           // aggregate reading the table: X, whose rows of newly discovered vertices it writes on the way (or null)
    const uint8_t *own;     // ... per edge, whether this edge is the one that writes it (null: the id map's entry carries its tag)
    MarkTag tag;            // ... how the id map's entries carry it
    int64_t ld_x;
    int64_t ld_src, ld_dst;
    uint64_t inv;
    uint32_t dimv;          // pieces per row ...
    uint32_t last;          // ... and the element at which the last one starts: the row's last four, which may overlap the piece before
    uint32_t rows;
    uint32_t max_fanout;
    int32_t vec4;           // rows are moved in pieces of four floats (else, below four, element by element)
    int32_t nt;             // aggregate inside a step: what it writes (means, rows of X) is stored past the caches (non-temporal)
    const int32_t *local_id; // aggregate that relabels its block's edges itself: the id map ...
    int32_t *col_out;        // ... and where col[e] = local id of nbr_gid[e] goes
    uint32_t blocks; // workgroups given to this role (0: role absent)
};

template <int VEC> struct VecOf;
template <> struct VecOf<4> {
    typedef v4f type;
    static __device__ __forceinline__ v4f zero() { return (v4f){0.0f, 0.0f, 0.0f, 0.0f}; }
};
template <> struct VecOf<1> {
    typedef float type;
    static __device__ __forceinline__ float zero() { return 0.0f; }
};

// "Gather": X[i,:] = feat[S[i],:].  A workgroup copies `rows` consecutive output rows; lanes walk the rows
// as one flat run of 16-byte pieces so that rows whose length is not a multiple of the wave width still
// fill every lane, four loads in flight per lane before the stores.
// (`s_row`: which of the workgroup's rows these are, if not all)
template <int VEC, bool STREAM, bool NT_STORE = false>
__device__ __forceinline__ void gather_rows(const RowArgs &a, uint32_t row0, uint32_t rows, const int32_t *s_id, const int32_t *s_row = nullptr)
{
    typedef typename VecOf<VEC>::type T;
    const uint32_t total = rows * a.dimv;
    for (uint32_t e0 = threadIdx.x; e0 < total; e0 += 4 * blockDim.x) {
        T val[4];
        uint32_t r[4], c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t e = e0 + u * blockDim.x;
            if (e < total) {
                r[u] = (uint32_t)(((uint64_t)e * a.inv) >> 32);
                c[u] = e - r[u] * a.dimv;
                const int32_t g = s_id[r[u]];
                c[u] = c[u] * VEC < a.last ? c[u] * VEC : a.last;
                const T *src = reinterpret_cast<const T *>(a.src + (int64_t)g * a.ld_src + c[u]);
                val[u] = g >= 0 ? (STREAM ? __builtin_nontemporal_load(src) : *src) : VecOf<VEC>::zero();
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t e = e0 + u * blockDim.x;
            if (e < total) {
                T *dst = reinterpret_cast<T *>(a.dst + (int64_t)(row0 + (s_row ? (uint32_t)s_row[r[u]] : r[u])) * a.ld_dst + c[u]);
                if (STREAM || NT_STORE)
                    __builtin_nontemporal_store(val[u], dst);
                else
                    *dst = val[u];
            }
        }
    }
}

// the frontier's rows only, beside the closing launch's ranking or ahead of a small step's aggregation
template <int VEC>
__device__ __forceinline__ void gather_rows_block(const RowArgs &a, uint32_t block, int32_t *s_id)
{
    const uint32_t n = *a.n_rows;
    const uint32_t row0 = block * a.rows;
    if (row0 >= n) return;
    const uint32_t rows = n - row0 < a.rows ? n - row0 : a.rows;
    if (threadIdx.x < rows) s_id[threadIdx.x] = a.S[row0 + threadIdx.x];
    __syncthreads();
    gather_rows<VEC, false, true>(a, row0, rows, s_id); // nothing in the step reads these rows of X again: stored past the caches
}

// ... without those the last hop reaches again, where its marks are bytes with tags: an edge to such a vertex reads its row for the mean and writes it
// into X on the way, as for a new vertex.  The vertex's entry gets the tag; its mark is this workgroup's to clear (the ranking
// tiles clear new vertices').  Saves reading the row, and costs the aggregation what it costs to write it (4.2 TB/s): worth it where the copy is longer than the
// ranking beside it by more than that, which both are bounds of.  us of the closing launch and the aggregation, all rows copied / these
// left out: 216 k rows of 2400 bytes 930 / 857, 706 k of 512 629 / 601, 722 k of 400 476 / 465, 622 k of 300 377 / 363, 125 k of 1 KB 185 / 175, 28 k
// of 2400 166 / 163, 33 k of 1 KB 80.2 / 78.0, 15 k of 2400 105.8 / 105.7; but 188 k rows of 400 bytes 156 / 163, 194 k of 256 115 / 117, 60 k of 400
// 67 / 70.  Hence by the frontier's bytes and the row's (reach_bytes), in the step's own sizes.  Where the lines lie: steps of one to four hops over eight
// graphs of 0.25 to 3 M vertices, in how many % the step is longer with all rows copied, mean (least, most):
//     rows of       34 MB              100 MB              140 MB              200 MB              300 MB              450 MB
//     300 to 400                       -2.2 (-4.1, 0.6)    -1.0 (-3.8, 5.0)    1.2 (-2.5, 9.5)     2.4 (-1.2, 7.3)     2.8 (0.0, 7.0)
//     512 to 768    0.3 (-0.9, 1.2)    0.3 (-2.4, 2.6)     0.7 (-3.3, 2.5)     1.4 (-2.7, 3.0)     2.9 (-1.0, 4.6)     4.5 (0.2, 6.4)
//     1000 to 2000  0.2 (-1.9, 1.6)    0.4 (-1.7, 2.7)     0.8 (-3.6, 3.3)     1.3 (-1.1, 4.4)     2.8 (0.8, 6.5)      4.0 (2.0, 6.2)
//     2048 to 2560  0.3 (-0.5, 1.3)    0.8 (-0.2, 2.3)     1.2 (0.3, 2.9)      1.4 (0.9, 1.9)      2.6 (1.7, 3.5)      4.0 (2.8, 5.2)
// What is slower above a line all the same: rows that end in partial lines, graphs of skew 0.9, where the copy finds its rows in the caches, and tables
// of the last-level cache's size.
template <int VEC>
__device__ __forceinline__ void gather_unreached_block(const RowArgs &a, uint32_t block, uint8_t *marks, int32_t *local_id, const MarkTag &tag, int32_t *s_mem)
{
    const uint32_t n = *a.n_rows;
    const uint32_t row0 = block * a.rows;
    if (row0 >= n) return;
    const uint32_t rows = n - row0 < a.rows ? n - row0 : a.rows;
    int32_t *const s_id = s_mem, *const s_row = s_mem + a.rows;
    uint32_t *const s_left = reinterpret_cast<uint32_t *>(s_row + a.rows);
    if (threadIdx.x == 0) *s_left = 0u;
    __syncthreads();
    if (threadIdx.x < rows) {
        const int32_t g = a.S[row0 + threadIdx.x];
        const uint32_t mark = g >= 0 ? marks[g] : 0u;
        if (mark) {
            marks[g] = 0;
            local_id[g] = tag.entry(row0 + threadIdx.x, mark);
        } else {
            const uint32_t at = atomicAdd(s_left, 1u);
            s_id[at] = g;
            s_row[at] = (int32_t)threadIdx.x;
        }
    }
    __syncthreads();
    gather_rows<VEC, false, true>(a, row0, *s_left, s_id, s_row);
}

// a launch of its own.  When the gathered matrix of this step is larger than the caches can hold for the aggregation that
// follows (decided on the device from the true row count), loads and stores are non-temporal: measured +15 % at 200 MB,
// -10 % at 90 MB.
template <int VEC>
__device__ __forceinline__ void gather_block(const RowArgs &a, uint32_t block, int32_t *s_id)
{
    const uint32_t n = *a.n_rows;
    const uint32_t row0 = block * a.rows;
    if (row0 >= n) return;
    const uint32_t rows = n - row0 < a.rows ? n - row0 : a.rows;
    if (threadIdx.x < rows) s_id[threadIdx.x] = a.S[row0 + threadIdx.x];
    __syncthreads();
    if ((uint64_t)n * a.dimv * (VEC * 4) > kGatherStreamBytes)
        gather_rows<VEC, true>(a, row0, rows, s_id);
    else
        gather_rows<VEC, false>(a, row0, rows, s_id);
}

// Launch l = 0..H of the hop kernel: it samples hop l for the rows of D_l (l < H) and, for l > 0, first ranks the
// vertices that hop l-1 discovered (they are the rows of D_l that D_{l-1} did not have).
struct HopArgs {
    const void *offsets;
    const int32_t *indices;
    Drmb *drmb;
    const Drmb *gate;
    StepInputs in;            // launch 0: the step's inputs ...
    const Mailbox *mailbox;   // ... or where it reads them itself (the gate owner's mailbox when gated)
    int32_t *S;
    int32_t *local_id;
    uint32_t *marks_prev;    // launches 1..H: the bitmap hop l-1 filled; ranked, consumed and cleared here
    uint32_t *marks_next;    // launches 0..H-1: the bitmap this launch's sampling fills
    uint32_t *seen;
    int32_t *row_ptr;         // block of hop l (launches 0..H-1)
    int32_t *nbr;
    uint8_t *own;             // last hop, when it marks bits and the aggregation writes X: per edge, whether it was the first to reach its vertex
    MarkTag tag;              // closing launch, when the last hop marked bytes and the aggregation writes X (see MarkTag)
    int32_t bytes_prev;       // marks_prev / marks_next hold a byte per vertex instead of a bit
    int32_t bytes_next;
    int32_t tag_next;         // the marks of this launch's sampling carry their edge's tag
    uint64_t *status_cnt;     // chained scans: vertices ranked, over the launch's ranking tiles ...
    uint64_t *status_edge;    // ... and edges sampled, over all its tickets
    uint32_t num_nodes;
    int32_t launch;           // l
    int32_t num_hops;         // H
    int32_t fanout;
    uint32_t rows_per_wave;   // rows whose slots a wavefront takes at a time: 64 / fanout
    uint32_t inv_fanout;      // lane / fanout == (lane * inv_fanout) >> 16 for lane < 64
    uint32_t rows_per_ticket; // old rows per ticket, at least
    uint32_t max_tickets;     // ... doubled until the launch's tickets stay within this (1024 rows at most)
    int32_t replace;
    uint32_t cap_rows;        // capacity of n_l
    uint32_t edge_cap;        // capacity of E_l
    uint32_t stage_edges;     // ids a workgroup holds in LDS between loading and storing them
    uint32_t words_per_tile;  // ranking tile (a multiple of 32)
    uint32_t chunk_log2;      // ... of at most a word per lane: a lane ranks 2^chunk_log2 vertices (4 .. 32)
    uint32_t rank_tiles;      // 0 for launch 0
    uint32_t batch;
    int32_t draw;             // tickets are drawn from a counter instead of being the workgroups' indices
    uint32_t patience;        // polls before a wait ends
    uint32_t blocks;          // workgroups of this role (the launch's first ones)
};

// LDS of a sampling workgroup of the hop kernel: up to 1024 rows of the block being sampled (vertex, degree, first edge
// offset, first edge), scan scratch; behind it (dynamic) the sampled ids on their way, the dedup set of a pass that marks
// bits, and a ranking tile's words
constexpr int kHopRows = kHopBlock; // one row per lane
struct HopShared {
    uint32_t drawn;
    uint32_t base_cnt;
    uint32_t base_edge;
    bool have_in;
    unsigned long long in[2];
    uint32_t wsum[64];                 // per round of the tile's words and wavefront: new vertices
    uint32_t wk[kHopBlock / 64];
    int32_t v[kHopRows];
    uint32_t deg[kHopRows], rp[kHopRows + 1];
    unsigned long long off[kHopRows];
};

constexpr uint32_t kMarkByte = 0x80u; // a vertex's mark byte: this bit, and the 7 low bits of the marking edge's index where tags are asked for

// which of four mark bytes are set, as the low four bits
__device__ __forceinline__ uint32_t marks4(uint32_t x) { return (((x >> 7) & 0x01010101u) * 0x10204080u) >> 28; }

// The slot positions of rows row0 .. row0 + 64/F - 1 of the workgroup's LDS rows, one wavefront: lane (r, j) = r F + j takes slot
// j of row row0 + r (vertex sh.v, degree sh.deg, first edge sh.rp): j itself if deg <= F, else Floyd's subset
// algorithm with one Philox draw per slot, all slots resolved at once (zg_floyd.h); with replacement one draw per slot.  Rows
// beyond `rows` and lanes beyond the last whole group take no slot.  Groups of F lanes instead of the next power of two: a
// wavefront holds 6 rows of fanout 10 instead of 4, 12 of fanout 5 instead of 8 - and Philox is what the pass computes most.
struct Slot {
    bool taken;
    uint32_t edge;          // its edge, counted from the batch's first
    unsigned long long src; // where its neighbor's id is
};

__device__ __forceinline__ Slot resolve_slot(const HopArgs &a, const HopShared &sh, uint32_t key_lo, uint32_t key_hi, uint32_t row0, uint32_t rows,
                                             int lane)
{
    const uint32_t F = (uint32_t)a.fanout;
    const uint32_t sub = ((uint32_t)lane * a.inv_fanout) >> 16;
    const uint32_t gl = (uint32_t)lane - sub * F;
    const uint32_t t = row0 + sub;
    const bool row = sub < a.rows_per_wave && t < rows;
    const uint32_t tl = row ? t : 0u;
    const int32_t tv = sh.v[tl];
    const uint32_t tdeg = row ? sh.deg[tl] : 0u;
    const bool slot = a.replace ? tdeg > 0u : gl < tdeg;
    uint32_t pos = gl;
    if (a.replace) {
        if (slot) pos = scale_draw(philox_draw(key_lo, key_hi, (uint32_t)a.launch, (uint32_t)tv, gl), tdeg);
    } else {
        const bool floyd = slot && tdeg > F;
        if (__any(floyd)) {
            uint32_t cand = gl;
            if (floyd) cand = scale_draw(philox_draw(key_lo, key_hi, (uint32_t)a.launch, (uint32_t)tv, gl), tdeg - F + gl + 1u);
            WaveGroup grp{sub * F};
            pos = floyd_position(grp, sub, gl, F, tdeg, floyd, cand);
        }
    }
    Slot r;
    r.edge = sh.rp[tl] + gl;
    r.taken = slot;
    r.src = sh.off[tl] + pos;
    return r;
}

// The neighbor ids of rows row0, row0 + step, .. (64/F rows at a time) below row_end into s_ids, by edge, edge e0 first; one wavefront.
// An id is stored only when the next slots have been worked out: its load is out for that long.
// A pass is bound by instruction issue (2 M edges: seven passes of 32 wavefronts per compute unit, 3 us each, the ids' loads 1 us of it):
// whole products in Philox, register moves instead of ds_bpermute in floyd_drawn_before and the loads' overlap took the hop launches from 23.4
// to 19.0 us (430 k edges), 18.0 to 16.3 (240 k), 14.5 to 14.0 (130 k); 54 us stay 54 at 2 M, where the random loads take over.
struct IdOut { // a load that is out: its id goes to s_ids[at]
    int32_t id;
    uint32_t at;
    bool out;
};

__device__ __forceinline__ IdOut load_ids(const HopArgs &a, const HopShared &sh, uint32_t key_lo, uint32_t key_hi, uint32_t row0, uint32_t row_end,
                                         uint32_t step, int lane, uint32_t e0, int32_t *s_ids)
{
    IdOut x = {0, 0u, false};
    for (; row0 < row_end; row0 += step) {
        const Slot slot = resolve_slot(a, sh, key_lo, key_hi, row0, row_end, lane);
        if (x.out) s_ids[x.at] = x.id;
        x.out = slot.taken;
        x.at = slot.edge - e0;
        if (x.out) x.id = a.indices[slot.src];
    }
    return x;
}

// Marks.  A hop that reaches many of the graph's vertices (bytes_next) stores a byte per sampled edge: idempotent stores
// need no dedup and no answer, and run at 50-150 G/s where atomics to the same addresses run at 12-25 G/s (2 M edges over 2.4 M
// vertices: 16 us against 86 us) and far slower on a hub's word.  The stores are plain byte stores, which the caches keep apart
// byte by byte; whichever of several edges' stores lands last, the byte says "reached", and nobody looks before the next
// launch.  (Stores that write through to memory at once queue up on a hub's byte like atomics: 129 -> 212 us in a launch of
// 2 M edges, against 81 us; a look at the byte first costs more than it spares, 84 us.)
// A hop that reaches few of them (a byte map of 110 M vertices made the closing launch 54 us longer) sets a bit, after a hash
// set in LDS: each distinct id of the pass reaches the hop's bitmap with at most one device-scope atomic - popular
// vertices are sampled hundreds of times per hop and same-address atomics serialise at the memory side.
// Ids that are already in D_l are marked too: the next launch masks them with "seen" (looking every id up in "seen" here was
// measured: one more dependent random load per edge, slower on every workload).
__device__ __forceinline__ void mark_byte(const HopArgs &a, uint32_t edge, int32_t g)
{
    if ((uint32_t)g < a.num_nodes)
        __hip_atomic_store(reinterpret_cast<uint8_t *>(a.marks_next) + (uint32_t)g, (uint8_t)(kMarkByte | (a.tag_next ? edge & 0x7Fu : 0u)),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void mark_bit(const HopArgs &a, uint32_t *set, uint32_t edge, int32_t g)
{
    bool mine = false;
    if ((uint32_t)g < a.num_nodes) {
        // first lane of the pass to insert g into the LDS set marks it (at most 1024 insertions into 2048 slots)
        uint32_t h = ((uint32_t)g * 2654435761u) >> (32 - kSampleHashBits);
        bool first = false;
        for (;;) {
            const uint32_t old = atomicCAS(&set[h], 0xFFFFFFFFu, (uint32_t)g);
            if (old == 0xFFFFFFFFu) {
                first = true;
                break;
            }
            if (old == (uint32_t)g) break;
            h = (h + 1) & (kSampleHashSlots - 1);
        }
        // The one atomic that finds the bit clear belongs to the first edge of the hop to reach the vertex.  For the last
        // hop that edge is remembered: the aggregation reads the vertex's feature row for it anyway and, if the vertex
        // turns out to be new, copies the row into X on the way (any one edge would do: they all carry the same row).
        if (first) {
            const uint32_t bit = 1u << (g & 31);
            if (a.own)
                mine = (atomicOr(&a.marks_next[(uint32_t)g >> 5], bit) & bit) == 0u;
            else
                atomicOr(&a.marks_next[(uint32_t)g >> 5], bit);
        }
    }
    if (a.own) a.own[edge] = mine ? 1 : 0;
}

__device__ __forceinline__ uint32_t row_length(const HopArgs &a, uint32_t deg)
{
    const uint32_t F = (uint32_t)a.fanout;
    return a.replace ? (deg > 0 ? F : 0u) : (deg < F ? deg : F);
}

// "Row lengths" of the workgroup's LDS rows: lane t takes the vertex sh.v[t] (none beyond `nrows`), loads its two offsets, and
// leaves degree and first edge offset in LDS.  Returns this lane's k = min(F, deg) (F whenever deg > 0 with replacement).
template <typename OffT>
__device__ __forceinline__ uint32_t load_rows(const HopArgs &a, HopShared &sh, uint32_t nrows, int tid)
{
    if ((uint32_t)tid >= nrows) return 0u;
    const int32_t v = sh.v[tid];
    uint32_t deg = 0;
    unsigned long long off0 = 0;
    if (v >= 0) {
        const OffT *off = (const OffT *)a.offsets;
        const OffT o0 = off[v], o1 = off[v + 1];
        off0 = (unsigned long long)o0;
        deg = (uint32_t)(o1 - o0);
    }
    sh.deg[tid] = deg;
    sh.off[tid] = off0;
    return row_length(a, deg);
}

// the same of any one vertex, the length alone
template <typename OffT>
__device__ __forceinline__ uint32_t vertex_length(const HopArgs &a, int32_t v)
{
    const OffT *off = (const OffT *)a.offsets;
    return row_length(a, (uint32_t)(off[v + 1] - off[v]));
}

// The same value in a scalar register of its own.  The compiler keeps some values that are the same for the whole workgroup in
// vector registers, and so all that it computes from them; and what a kernel's head and its tail compute alike it computes once, at the
// head, and keeps: registers of which k_hop has none to spare (they go to memory).
__device__ __forceinline__ int32_t own_scalar(int32_t x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// ... and a vector register
__device__ __forceinline__ uint32_t own_vector(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// the lowest q set bits of x
__device__ __forceinline__ uint32_t lowest_set_bits(uint32_t x, uint32_t q)
{
    uint32_t out = 0;
    while (x && q) {
        const uint32_t low = x & (0u - x);
        out |= low;
        x ^= low;
        --q;
    }
    return out;
}

// The hop kernel's launches 0 .. H-1 (k_hop) and the closing launch H (k_close).  Every workgroup has a ticket; in ticket
// order a launch's work is the row order of block l:
//   tickets 0 .. t_old-1   rows that were already in D_{l-1} (launch 0: the seeds);
//   then the ranking tiles of hop l-1's marks, 32 W vertices each, in ascending vertex id: those marked and not "seen"
//                          are the hop's new vertices; their rank - n_{l-1} plus the new vertices before them - is
//                          their local id and their row in block l, so they land behind D_{l-1} in ascending id.
// Two single-pass chained scans run over the tickets: new vertices and sampled edges.  A ticket first finds its rows'
// lengths k_i = min(F, deg) ("row lengths"; a row per lane, 1024 at a time, held in LDS), publishes both totals, takes its
// exclusive prefixes (wavefront 0 and wavefront 1, side by side), and then writes S, the id map and row_ptr ("offsets
// scan") and samples its rows, F lanes per row ("sample").  New vertices join "seen", consumed marks are cleared.  Vertices
// ranked beyond the cap are dropped (no row, local id -1, not "seen") and the hop's overflow bit is raised; the rows kept are
// a prefix of the row order, so the block stays consistent up to the cap.  Launch H ranks only.  The launch's surplus
// workgroups (the grid is sized by the caps) have no ticket and return.
//
// A ticket is the workgroup's index, or drawn from a counter (HopArgs.draw).  Drawing costs: the counter answers once per 13 ns, so the
// last of 240 workgroups has its ticket 5.7 us into the launch, the last of 470 after 9.4 (large launches with one plan 20.3 -> 16.5 us, 53.7 -> 46,
// launch 0 12.4 -> 8.1 with 128 of them).  It pays where the chip is shared: a workgroup that starts late, because another stream's kernels
// hold its place, gets a late ticket, while a late index keeps all those behind it waiting in places that others could use (110 M
// vertices, four plans: 217 us per step drawn, 235 by index; one plan 251-270 / 250-260).  With smaller graphs it pays little or nothing even
// there.  us per step drawn / by index: 2.4 M vertices and 115 M edges, three hops, one plan 102.6 / 94.9, two on two streams 80.9 /
// 78.3, four 85.6 / 84.0, beside a matrix product on another stream 219 / 213, beside a copy 226 / 221; sampling alone 120.7 / 112.7, 98.0 /
// 95.7, 103.1 / 100.5, 227 / 219, 209 / 205; 1 M vertices and hubs 100.1 / 96.4, 91.4 / 89.5, 92.3 / 91.1; the benchmark's smaller workloads, four
// plans: 52.3 / 52.6 (large_sparse), 68.4 / 68.9 (medium_dense), 62.6 / 64.3 (envelope_stress), and 87.9 / 83.8, 95.1 / 93.5, 87.2 / 83.6 with one.  So tiles
// that are ranked by pieces of 128 vertices (of more than a word per lane: long launches, with nobody who could work out a missing
// total) draw, and no other launch does.
//
// Bound by latency: a ticket is a chain of about eight dependent memory accesses, so a launch costs the length of that chain,
// the code it walks through cold and its slowest ticket.  Hence one instantiation per kind of launch and of marks (one
// kernel for all spilled 140 scalar and 6 vector registers) and wide scans in registers.

// The words of a ranking tile, bit b of word w: vertex 32 w + b is marked and not "seen".  A lane holds pieces of four words,
// piece u NT + tid in round u: 16-byte accesses, consecutive lanes consecutive.
__device__ __forceinline__ uint32_t piece_word(const uint4 &x, uint32_t c) { return c == 0 ? x.x : c == 1 ? x.y : c == 2 ? x.z : x.w; }
__device__ __forceinline__ uint32_t piece_any(const uint4 &x) { return x.x | x.y | x.z | x.w; }

// the marks of one word's 32 bytes
__device__ __forceinline__ uint32_t marks32(const uint4 *b)
{
    const uint4 y = b[0], z = b[1];
    return marks4(y.x) | (marks4(y.y) << 4) | (marks4(y.z) << 8) | (marks4(y.w) << 12) | (marks4(z.x) << 16) | (marks4(z.y) << 20) | (marks4(z.z) << 24) |
           (marks4(z.w) << 28);
}

// Reads a tile's marks, masks them with "seen", and clears them for the hop after next (tagged: a new vertex's byte stays until
// its tag has been read; with `reach` a frontier vertex's byte is the copy's to clear).  Mark bytes become words in LDS first, 16 bytes per lane.  With JOIN the new vertices join
// "seen" at once: this workgroup is its words' only reader and writer in the launch.  The loads of all rounds are on their
// way before the first is looked at, and so are the words of "seen".
template <int NT, int R, bool BYTES, bool JOIN>
__device__ __forceinline__ void load_tile(const HopArgs &a, size_t tile0, uint32_t np, uint32_t tid, uint4 (&x)[R], uint32_t *s_words, bool reach = false)
{
    uint4 *src = reinterpret_cast<uint4 *>(a.marks_prev) + (BYTES ? tile0 * 2u : tile0 / 4u), *seen = reinterpret_cast<uint4 *>(a.seen + tile0);
    if (BYTES) {
        uint16_t *half = reinterpret_cast<uint16_t *>(s_words);
#pragma unroll 4
        for (uint32_t q = tid; q < 8u * np; q += (uint32_t)NT) {
            const uint4 y = src[q];
            half[q] = (uint16_t)(marks4(y.x) | (marks4(y.y) << 4) | (marks4(y.z) << 8) | (marks4(y.w) << 12));
        }
        __syncthreads();
    }
    uint4 sn[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const uint32_t q = u * (uint32_t)NT + tid;
        x[u] = make_uint4(0u, 0u, 0u, 0u);
        if (q < np) x[u] = BYTES ? reinterpret_cast<const uint4 *>(s_words)[q] : src[q];
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (piece_any(x[u])) sn[u] = seen[u * (uint32_t)NT + tid];
    const bool tagged = BYTES && !JOIN && a.tag.shift != 0;
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (piece_any(x[u])) {
            const uint32_t q = u * (uint32_t)NT + tid;
            const uint4 marked = x[u];
            x[u].x &= ~sn[u].x, x[u].y &= ~sn[u].y, x[u].z &= ~sn[u].z, x[u].w &= ~sn[u].w;
            if (JOIN && piece_any(x[u])) seen[q] = make_uint4(sn[u].x | x[u].x, sn[u].y | x[u].y, sn[u].z | x[u].z, sn[u].w | x[u].w);
            if (!BYTES) {
                src[q] = make_uint4(0u, 0u, 0u, 0u);
            } else if (JOIN || !reach) {
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c) {
                    const uint32_t w = piece_word(marked, c), fresh = piece_word(x[u], c);
                    uint4 *b = src + 2u * (4u * q + c); // the word's 32 bytes
                    if (w && (!tagged || fresh == 0u))
                        b[0] = b[1] = make_uint4(0u, 0u, 0u, 0u);
                    else
                        for (uint32_t old = w & ~fresh; old; old &= old - 1u) reinterpret_cast<uint8_t *>(b)[__ffs((int)old) - 1] = 0;
                }
            }
        }
}

// a word of a tile: its marks, and those of new vertices
struct TileWord {
    uint32_t marked, fresh;
};

// Clears a word's marks for the hop after next; where tags are still needed (`tagged`) a new vertex's byte stays until its tag has been read.
template <bool BYTES>
__device__ __forceinline__ void clear_marks(const HopArgs &a, size_t word, TileWord x, bool tagged)
{
    uint4 *const bytes = reinterpret_cast<uint4 *>(a.marks_prev) + word * 2u;
    if (!BYTES)
        a.marks_prev[word] = 0u;
    else if (!tagged || x.fresh == 0u)
        bytes[0] = bytes[1] = make_uint4(0u, 0u, 0u, 0u);
    else
        for (uint32_t old = x.marked & ~x.fresh; old; old &= old - 1u) reinterpret_cast<uint8_t *>(bytes)[__ffs((int)old) - 1] = 0;
}

// a word of a tile, whoever's it is: marked and not "seen" (rarely needed, and in few registers)
template <bool BYTES>
__device__ __forceinline__ uint32_t new_vertices(const HopArgs &a, uint32_t word)
{
    uint32_t w = 0u;
    if (BYTES) {
#pragma unroll 1
        for (uint32_t c = 0; c < 8u; ++c) w |= marks4(a.marks_prev[(size_t)word * 8u + c]) << (4u * c);
    } else {
        w = a.marks_prev[word];
    }
    return w & ~a.seen[word];
}

// a tile's total, worked out by one wavefront of another workgroup (see chain_prefix)
template <bool BYTES>
__device__ __forceinline__ uint32_t missing_vertices(const HopArgs &a, uint32_t tile, uint32_t lane)
{
    const uint32_t w0 = tile * a.words_per_tile;
    uint32_t c = 0;
#pragma unroll 1
    for (uint32_t w = lane; w < a.words_per_tile; w += 64u) c += __popc(new_vertices<BYTES>(a, w0 + w));
    return wave_sum(c);
}

// Ranks within the tile: lex[u] = new vertices before the lane's piece of round u.  Returns their number.  `wsum` holds a count
// per round and wavefront (64 at most); one barrier.
template <int NT, int R>
__device__ __forceinline__ uint32_t rank_pieces(const uint4 (&x)[R], uint32_t (&lex)[R], uint32_t *wsum, uint32_t np, uint32_t wave, uint32_t lane)
{
    constexpr uint32_t NW = NT / 64;
    static_assert(R * NW <= 64, "one count per lane");
    uint32_t rounds = 0;
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (u * (uint32_t)NT < np) {
            const uint32_t c = __popc(x[u].x) + __popc(x[u].y) + __popc(x[u].z) + __popc(x[u].w), incl = wave_incl_scan(c);
            if (lane == 63u) wsum[u * NW + wave] = incl;
            lex[u] = incl - c;
            rounds = u + 1u;
        }
    __syncthreads();
    const uint32_t e = lane < rounds * NW ? wsum[lane] : 0u;
    const uint32_t s = wave_incl_scan(e);
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (u * (uint32_t)NT < np) lex[u] += lane_value(s, u * NW + wave) - lane_value(e, u * NW + wave);
    return lane_value(s, 63u);
}

// the new vertices number c0 .. c0 + n - 1 of the tile into v
__device__ __forceinline__ void expand_piece(const uint4 &x, uint32_t j, uint32_t first_word, uint32_t c0, uint32_t n, int32_t *v)
{
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c)
        for (uint32_t w = piece_word(x, c); w; w &= w - 1u, ++j)
            if (j - c0 < n) v[j - c0] = (int32_t)(((first_word + c) << 5) + (uint32_t)__ffs((int)w) - 1u);
}

// A tile of at most a word per lane (the graph is small for its ranking tiles, the tile dense with new vertices): the lane's word
// of marks and of new vertices, the latter also left in s_words.  A word per lane while it is read, and 2^chunk_log2 vertices per lane once it is ranked and
// expanded (pieces of 128 left 16 lanes of 1024 to walk through a tile of 64 words, up to 128 vertices one after another: a hop launch
// over 250 k vertices 15.6 -> 14.5 us, with 2.4 M vertices 57 -> 54).
template <int NT, bool BYTES>
__device__ __forceinline__ TileWord load_words(const HopArgs &a, size_t tile0, uint32_t words, uint32_t tid, uint32_t *s_words)
{
    uint32_t sn = 0u, marked = 0u;
    if (tid < words) sn = a.seen[tile0 + tid];
    if (BYTES) {
        const uint4 *src = reinterpret_cast<const uint4 *>(a.marks_prev) + tile0 * 2u;
        uint16_t *half = reinterpret_cast<uint16_t *>(s_words);
#pragma unroll 2
        for (uint32_t q = tid; q < 2u * words; q += (uint32_t)NT) {
            const uint4 y = src[q];
            half[q] = (uint16_t)(marks4(y.x) | (marks4(y.y) << 4) | (marks4(y.z) << 8) | (marks4(y.w) << 12));
        }
        __syncthreads();
        if (tid < words) marked = s_words[tid];
    } else if (tid < words) {
        marked = a.marks_prev[tile0 + tid];
    }
    if (tid < words) s_words[tid] = marked & ~sn;
    return {marked, marked & ~sn};
}

// ... and what changes once the tile's totals are published: its marks are cleared - read again: no register of k_hop holds them that long -
// and its new vertices join "seen".
template <bool BYTES>
__device__ __forceinline__ void settle_word(const HopArgs &a, size_t tile0, uint32_t words, uint32_t tid, const uint32_t *s_words)
{
    if (tid >= words) return;
    const uint32_t marked = BYTES ? marks32(reinterpret_cast<uint4 *>(a.marks_prev) + (tile0 + tid) * 2u) : a.marks_prev[tile0 + tid], fresh = s_words[tid];
    if (fresh) a.seen[tile0 + tid] |= fresh;
    if (marked) clear_marks<BYTES>(a, tile0 + tid, {marked, fresh}, false);
}

// ... and its ranks: the lane's chunk of the tile's words (in s_words: barriers before the first and after the last use are in
// here), `before` = new vertices ahead of it.  Returns their number.  `wsum` holds a count per wavefront.
template <int NT>
__device__ __forceinline__ uint32_t rank_chunks(uint32_t word, uint32_t chunk_log2, uint32_t words, const uint32_t *s_words, uint32_t *wsum, uint32_t tid,
                                                uint32_t &chunk, uint32_t &before)
{
    const uint32_t lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    __syncthreads();
    chunk = word;
    if (chunk_log2 < 5u) {
        const uint32_t at = tid << chunk_log2, w = at >> 5;
        chunk = w < words ? (s_words[w] >> (at & 31u)) & ((1u << (1u << chunk_log2)) - 1u) : 0u;
    }
    const uint32_t c = __popc(chunk), incl = wave_incl_scan(c);
    if (lane == 63u) wsum[wave] = incl;
    __syncthreads();
    const uint32_t e = lane < (uint32_t)NT / 64u ? wsum[lane] : 0u, sum = wave_incl_scan(e);
    before = lane_value(sum, wave) - lane_value(e, wave) + incl - c;
    return lane_value(sum, 63u);
}

// the new vertices number c0 .. c0 + n - 1 of the tile into v: those of one chunk, the first of which is vertex `first`
__device__ __forceinline__ void expand_chunk(uint32_t chunk, uint32_t before, uint32_t first, uint32_t c0, uint32_t n, int32_t *v)
{
    for (uint32_t j = before - c0; chunk; chunk &= chunk - 1u, ++j)
        if (j < n) v[j] = (int32_t)(first + (uint32_t)__ffs((int)chunk) - 1u);
}

struct HopRoles { // the other workgroups of launches 0 .. H-1
    RelabelArgs rel; // launches 2 ..
    IngestArgs ing;  // launch 0
};

template <typename OffT, bool FIRST, bool PREV_BYTES, bool NEXT_BYTES>
__global__ __launch_bounds__(kHopBlock, 8) void k_hop(HopArgs a, HopRoles o)
{
    constexpr int R = (PREV_BYTES ? kHopMaxTileWords : kHopFatTileWords) / 4 / kHopBlock; // rounds of a tile
    __shared__ HopShared sh;
    extern __shared__ __align__(16) uint32_t s_dyn[]; // the sampled ids on their way, the dedup set of a bit-marking pass, a ranking tile's words
    if (gate_closed(a.gate)) return;
    // roles by workgroup index: the tickets, then the ingest or relabel role
    if (blockIdx.x >= a.blocks) {
        if (FIRST)
            ingest_block(o.ing, blockIdx.x - a.blocks, sh.in);
        else
            relabel_block(o.rel, blockIdx.x - a.blocks);
        return;
    }
    int32_t *const s_ids = reinterpret_cast<int32_t *>(s_dyn);
    uint32_t *const s_set = s_dyn + a.stage_edges;
    uint32_t *const s_words = s_set + (NEXT_BYTES ? 0 : kSampleHashSlots);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    Drmb *d = a.drmb;
    const bool by_mail = FIRST && !a.in.seeds;
    if (by_mail && tid == 64) sh.have_in = prefetched_inputs(d, a.gate, sh.in);
    if (!FIRST && a.draw && tid == 0) sh.drawn = atomicAdd(&d->ticket[a.launch], 1u);
    const uint32_t n_old_d = FIRST ? a.batch : d->n[a.launch - 1]; // (in flight while a drawn ticket comes back)
    const uint32_t key_lo_d = FIRST ? 0u : d->key_lo, key_hi_d = FIRST ? 0u : d->key_hi;
    uint32_t ticket = blockIdx.x;
    if (by_mail || (!FIRST && a.draw)) {
        __syncthreads();
        if (!FIRST) ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.drawn);
    }
    // A scalar, and with it all that follows from it (rows per ticket, the tile, its address, which kind of ticket this is): kept per lane
    // these cost a launch that marks bits 7 registers more than its 64, 28 bytes per lane written to scratch - 14 MB in a launch of
    // 480 tickets.  (110 M vertices: 88 + 38 MB read + written by that launch, now 79 + 24 MB; the step 280 -> 274 us.)
    const uint32_t n_old = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_old_d);
    // old rows per ticket: more than the plan's when there are so many that the launch would need a second round of workgroups
    uint32_t rows = a.rows_per_ticket;
    if (!FIRST && rows < 128u) rows = 128u;
    if (!FIRST)
        while (rows < (uint32_t)kHopRows / 2u + 1u && (n_old + rows - 1u) / rows + a.rank_tiles > a.max_tickets) rows *= 2u;
    const uint32_t t_old = (uint32_t)__builtin_amdgcn_readfirstlane((int)((n_old + rows - 1u) / rows));
    const uint32_t n_tickets = t_old + (FIRST ? 0u : a.rank_tiles);
    if (ticket >= n_tickets) return;
    if (by_mail && !sh.have_in) {
        if (tid == 0) shared_inputs(d, a.gate, a.mailbox, ticket, a.patience, sh.in);
        __syncthreads();
    }
    const unsigned long long seeds_at = by_mail ? sh.in[0] : (unsigned long long)a.in.seeds, key = by_mail ? sh.in[1] : a.in.key; // (launch 0)
    const bool old = FIRST || ticket < t_old; // uniform over the workgroup
    const uint32_t key_lo = FIRST ? (uint32_t)(key & 0xFFFFFFFFull) : key_lo_d;
    const uint32_t key_hi = FIRST ? (uint32_t)(key >> 32) : key_hi_d;

    // ---- what this ticket's rows are: m old rows from r0 on, or the tile's m new vertices
    uint32_t m;
    const uint32_t r0 = ticket * rows, tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)(ticket - t_old));
    const uint32_t np = a.words_per_tile / 4u; // the tile's pieces
    const size_t tile0 = (size_t)tile * a.words_per_tile;
    uint4 *const s_piece = reinterpret_cast<uint4 *>(s_words);
    const bool by_chunks = a.words_per_tile <= (uint32_t)kHopBlock;
    auto rank_and_expand = [&](uint32_t word, uint32_t c0, bool publish) { // by chunks
        uint32_t chunk, before;
        const uint32_t t = own_vector(tid);
        const uint32_t n = rank_chunks<kHopBlock>(word, a.chunk_log2, a.words_per_tile, s_words, sh.wsum, t, chunk, before);
        if (publish && tid == 0) chain_publish(a.status_cnt, tile, n);
        expand_chunk(chunk, before, ((uint32_t)tile0 << 5) + (t << a.chunk_log2), c0, kHopRows, sh.v);
        return n;
    };
    auto expand_pieces = [&](const uint4 (&x)[R], const uint32_t (&lex)[R], uint32_t c0, uint32_t t) {
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (u * (uint32_t)kHopBlock + t < np) expand_piece(x[u], lex[u], (uint32_t)tile0 + (u * (uint32_t)kHopBlock + t) * 4u, c0, kHopRows, sh.v);
    };
    // the tile's words as they were ranked, out of LDS, and their ranks once more: no register holds them (a tile of several batches of
    // rows, or cut by the cap)
    auto pieces_again = [&](uint4 (&x)[R], uint32_t (&lex)[R], uint32_t t) {
#pragma unroll
        for (int u = 0; u < R; ++u) x[u] = u * (uint32_t)kHopBlock + t < np ? s_piece[u * kHopBlock + t] : make_uint4(0u, 0u, 0u, 0u);
        (void)rank_pieces<kHopBlock, R>(x, lex, sh.wsum, np, wave, lane);
    };
    if (old) {
        m = n_old - r0 < rows ? n_old - r0 : rows;
    } else if (by_chunks) {
        m = rank_and_expand(load_words<kHopBlock, PREV_BYTES>(a, tile0, a.words_per_tile, tid, s_words).fresh, 0u, true);
    } else {
        uint4 x[R];
        uint32_t lex[R];
        load_tile<kHopBlock, R, PREV_BYTES, true>(a, tile0, np, tid, x, s_words);
        m = rank_pieces<kHopBlock, R>(x, lex, sh.wsum, np, wave, lane);
        if (tid == 0) chain_publish(a.status_cnt, tile, m);
        expand_pieces(x, lex, 0u, tid);
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (u * (uint32_t)kHopBlock + tid < np) s_piece[u * kHopBlock + tid] = x[u]; // (read back by this lane only)
    }
    auto old_row = [&](uint32_t r) { // a row of the frontier (launch 0: a seed, an out-of-range one becoming -1, a vertex without neighbors)
        const int32_t v = FIRST ? reinterpret_cast<const int32_t *>(seeds_at)[r] : a.S[r];
        return FIRST && (uint32_t)v >= a.num_nodes ? -1 : v;
    };
    auto missing_edges = [&](uint32_t t) { // another ticket's edges, worked out by this wavefront (see chain_prefix)
        uint32_t k = 0;
        if (t < t_old) {
#pragma unroll 1
            for (uint32_t i = lane; i < rows && t * rows + i < n_old; i += 64u) {
                const int32_t v = old_row(t * rows + i);
                if (v >= 0) k += vertex_length<OffT>(a, v);
            }
        } else if (!FIRST) {
            const uint32_t w0 = (t - t_old) * a.words_per_tile;
#pragma unroll 1
            for (uint32_t w = lane; w < a.words_per_tile; w += 64u)
#pragma unroll 1
                for (uint32_t x = new_vertices<PREV_BYTES>(a, w0 + w); x; x &= x - 1u) k += vertex_length<OffT>(a, (int32_t)((w0 + w) * 32u) + __ffs((int)x) - 1);
        }
        return wave_sum(k);
    };

    // rows c0 .. c0 + 1023 of the ticket into sh.v: old rows from the frontier list, new vertices expanded from the tile's words
    // (`first`: a tile's first batch has been there since it was ranked)
    auto fill_rows = [&](uint32_t c0, bool first) {
        if (old) {
            if (tid < m) sh.v[tid] = old_row(r0 + tid);
        } else if (!first && by_chunks) {
            (void)rank_and_expand(tid < a.words_per_tile ? s_words[tid] : 0u, c0, false);
        } else if (!first) {
            uint4 x[R];
            uint32_t lex[R];
            const uint32_t t = own_vector(tid);
            pieces_again(x, lex, t);
            expand_pieces(x, lex, c0, t);
        }
        __syncthreads();
    };

    // ---- row lengths, a row per lane; their total goes into the edge chain
    const uint32_t supers = (m + kHopRows - 1) / kHopRows;
    uint32_t k = 0, kincl = 0; // this lane's row's length and the wavefront's sum up to it (of the last batch of rows)
    {
        uint32_t before = 0; // earlier batches
        for (uint32_t q = 0; q < supers; ++q) {
            const uint32_t c0 = q * kHopRows;
            fill_rows(c0, q == 0);
            before += lane_value(kincl, 63u);
            k = load_rows<OffT>(a, sh, m - c0 < (uint32_t)kHopRows ? m - c0 : (uint32_t)kHopRows, tid);
            kincl = wave_incl_scan(k);
            if (q + 1 < supers) __syncthreads(); // the next fill overwrites sh.v
        }
        if (lane == 63u) sh.wk[wave] = before + kincl;
    }
    __syncthreads();
    uint32_t wk = lane < (uint32_t)kHopBlock / 64u ? sh.wk[lane] : 0u, wks = wave_incl_scan(wk);
    const uint32_t ticket_edges = lane_value(wks, 63u);
    if (tid == 0) chain_publish(a.status_edge, ticket, ticket_edges);

    // ---- sample and offsets scan, a batch of 1024 rows at a time, as many of them at once as their ids fit into LDS.  A single
    // batch is still in LDS from above; several are redone (their loads hit the cache).  The first ids are loaded
    // before the chains are asked for: what a ticket waits for longest - the ids, out of an array of gigabytes, and the
    // tickets before it - it waits for once.  Marks are set behind the chains: rows beyond the cap leave none.
    const uint32_t rpw = a.rows_per_wave, step = rpw * (uint32_t)(kHopBlock / 64);
    const uint32_t stage_rows = a.stage_edges / (uint32_t)a.fanout;
    uint32_t rank0 = r0, room = 0xFFFFFFFFu, ebase = 0;
    bool chained = false;
    auto take_prefixes = [&]() { // wavefront 0 sums up the new vertices before this tile, wavefront 1 the edges before this ticket
        if (wave == 0u && !old) {
            const uint32_t c = chain_prefix<FIRST ? 4 : 1>(a.status_cnt, tile, m, d, (int)lane, a.patience, [&](uint32_t t) { return missing_vertices<PREV_BYTES>(a, t, lane); });
            if (lane == 0) sh.base_cnt = c;
        }
        if (wave == 1u) {
            const uint32_t e = chain_prefix<FIRST ? 4 : 1>(a.status_edge, ticket, ticket_edges, d, (int)lane, a.patience, missing_edges);
            if (lane == 0) sh.base_edge = e;
        }
    };
    auto use_prefixes = [&]() {
        if (!old) rank0 = n_old + (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.base_cnt); // row index of the ticket's first row
        room = rank0 < a.cap_rows ? a.cap_rows - rank0 : 0u;                                  // how many of its rows fit (old rows: all)
        ebase = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.base_edge);
        chained = true;
    };
    for (uint32_t q = 0; q == 0u || q < supers; ++q) { // (a tile without a new vertex: once, for the prefixes)
        const uint32_t c0 = q * kHopRows;
        const uint32_t nrows = m - c0 < (uint32_t)kHopRows ? m - c0 : (uint32_t)kHopRows;
        if (supers > 1) {
            if (q) __syncthreads(); // the last batch's rows have been read
            fill_rows(c0, false);
            k = load_rows<OffT>(a, sh, nrows, tid);
            kincl = wave_incl_scan(k);
            if (lane == 63u) sh.wk[wave] = kincl;
            __syncthreads();
            wk = lane < (uint32_t)kHopBlock / 64u ? sh.wk[lane] : 0u;
            wks = wave_incl_scan(wk);
        }
        const uint32_t batch_edges = lane_value(wks, 63u);
        if (tid < nrows) sh.rp[tid] = lane_value(wks, wave) - lane_value(wk, wave) + kincl - k;
        if (tid == 0) sh.rp[nrows] = batch_edges;
        __syncthreads();
        uint32_t keep = 0;
        for (uint32_t b0 = 0; b0 == 0u || b0 < nrows; b0 += stage_rows) {
            const uint32_t b1 = b0 + stage_rows < nrows ? b0 + stage_rows : nrows, e0 = sh.rp[b0];
            const IdOut last = load_ids(a, sh, key_lo, key_hi, b0 + wave * rpw, b1, step, (int)lane, e0, s_ids);
            if (!chained) take_prefixes(); // (while the last id is on its way)
            if (last.out) s_ids[last.at] = last.id;
            __syncthreads();
            if (!chained) use_prefixes();
            keep = room > c0 ? (room - c0 < nrows ? room - c0 : nrows) : 0u; // dropped rows sample nothing
            const uint32_t e1 = keep > b0 ? sh.rp[keep < b1 ? keep : b1] : e0;
            if (NEXT_BYTES) {
                for (uint32_t e = e0 + tid; e < e1; e += (uint32_t)kHopBlock) {
                    const uint32_t edge = ebase + e;
                    if (edge < a.edge_cap) {
                        const int32_t g = s_ids[e - e0];
                        a.nbr[edge] = g;
                        mark_byte(a, edge, g);
                    }
                }
            } else {
                for (uint32_t f = e0; f < e1; f += (uint32_t)kHopBlock) {
                    for (uint32_t x = tid; x < (uint32_t)kSampleHashSlots; x += (uint32_t)kHopBlock) s_set[x] = 0xFFFFFFFFu;
                    __syncthreads();
                    const uint32_t e = f + tid, edge = ebase + e;
                    if (e < e1 && edge < a.edge_cap) {
                        const int32_t g = s_ids[e - e0];
                        a.nbr[edge] = g;
                        mark_bit(a, s_set, edge, g);
                    }
                    if (f + (uint32_t)kHopBlock < e1) __syncthreads(); // the set is reset by the next pass
                }
            }
            if (b1 < nrows) __syncthreads(); // the ids and the set are reused
        }
        if (tid < nrows) {
            const int32_t gid = sh.v[tid];
            if (tid < keep) {
                a.row_ptr[rank0 + c0 + tid] = (int32_t)(ebase + sh.rp[tid]);
                if (!old) {
                    a.S[rank0 + c0 + tid] = gid;
                    a.local_id[gid] = (int32_t)(rank0 + c0 + tid);
                }
            } else {
                a.local_id[gid] = -1;
            }
        }
        ebase += sh.rp[keep];
    }
    if (old) {
        if (FIRST && ticket == t_old - 1u && tid == 0) { // launch 0 has no ranking tiles: the block ends with these rows
            a.row_ptr[n_old] = (int32_t)ebase;
            d->E[a.launch] = ebase;
        }
        return;
    }

    const uint32_t tid_end = own_vector(tid);
    if (by_chunks) settle_word<PREV_BYTES>(a, tile0, a.words_per_tile, tid_end, s_words);

    if (m > room) {
        // ---- the cap cuts into this tile: the vertices dropped leave "seen" again
        uint4 x[R];
        uint32_t lex[R];
        __syncthreads();
        pieces_again(x, lex, tid_end);
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (u * (uint32_t)kHopBlock + tid_end < np) {
                uint32_t j = lex[u];
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c) {
                    const uint32_t w = piece_word(x[u], c), pc = __popc(w);
                    const uint32_t kept = j < room ? lowest_set_bits(w, room - j) : 0u;
                    if (kept != w) a.seen[tile0 + (u * (uint32_t)kHopBlock + tid_end) * 4u + c] &= ~(w & ~kept);
                    j += pc;
                }
            }
    }

    // ---- end of the block: the tile in which the cap falls closes a truncated block; the last ticket publishes the
    // hop's sizes and, when everything fitted, closes the block
    if (tid == 0) {
        const int32_t launch = own_scalar(a.launch);
        if (rank0 <= a.cap_rows && (uint64_t)rank0 + m > a.cap_rows) {
            a.row_ptr[a.cap_rows] = (int32_t)ebase;
            d->E[launch] = ebase;
        }
        if (ticket == n_tickets - 1u) {
            const uint64_t exact = (uint64_t)rank0 + m;
            d->n_exact[launch] = (uint32_t)exact;
            d->n[launch] = exact < a.cap_rows ? (uint32_t)exact : a.cap_rows;
            if (exact > a.cap_rows) {
                atomicOr(&d->flags, ZG_FLAG_HOP_OVERFLOW(launch - 1));
                atomicOr(&d->step_flags, ZG_FLAG_HOP_OVERFLOW(launch - 1));
            } else {
                a.row_ptr[exact] = (int32_t)ebase;
                d->E[launch] = ebase;
            }
        }
    }
}

// A small step's sampling, all hops of it in one workgroup: what the hop launches do, with the marks and "seen" as bitmaps in
// LDS and barriers where they have launches and chained scans.  Outputs are the same; the global marks, "seen" and scan state
// stay zero.  The last hop is relabeled by the launch that follows, the others here.
struct SmallArgs {
    HopArgs hop;     // what does not depend on the hop
    int32_t *row_ptr[ZG_MAX_HOPS], *nbr[ZG_MAX_HOPS], *col[ZG_MAX_HOPS];
    uint32_t fanout[ZG_MAX_HOPS], edge_cap[ZG_MAX_HOPS];
    uint32_t cap[ZG_MAX_HOPS + 1];
    uint32_t words;  // of a bitmap, a multiple of 32
};

template <typename OffT>
__global__ __launch_bounds__(kHopBlock) void k_small(SmallArgs s)
{
    constexpr int R = kSmallMaxWords / 4 / kHopBlock; // rounds of a bitmap's pieces
    __shared__ HopShared sh;
    extern __shared__ __align__(16) uint32_t s_dyn[]; // the sampled ids on their way, the hop's marks, "seen"
    if (gate_closed(s.hop.gate)) return;
    HopArgs a = s.hop;
    int32_t *const s_ids = reinterpret_cast<int32_t *>(s_dyn);
    uint32_t *const s_marks = s_dyn + a.stage_edges, *const s_seen = s_marks + s.words;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    Drmb *d = a.drmb;
    if (!a.in.seeds && tid == 0 && !prefetched_inputs(d, a.gate, sh.in)) mailbox_inputs(d, a.gate, a.mailbox, sh.in);
    for (uint32_t w = tid; w < 2u * s.words; w += (uint32_t)kHopBlock) s_marks[w] = 0u;
    __syncthreads();
    const int32_t *seeds = a.in.seeds ? a.in.seeds : reinterpret_cast<const int32_t *>(sh.in[0]);
    const unsigned long long key = a.in.seeds ? a.in.key : sh.in[1];
    const uint32_t key_lo = (uint32_t)(key & 0xFFFFFFFFull), key_hi = (uint32_t)(key >> 32);
    if (tid == 0) {
        d->step = d->epoch;
        d->n[0] = a.batch;
        d->n_exact[0] = a.batch;
        d->key_lo = key_lo;
        d->key_hi = key_hi;
    }
    for (uint32_t i = tid; i < a.batch; i += (uint32_t)kHopBlock) {
        int32_t v = seeds[i];
        if ((uint32_t)v >= a.num_nodes) {
            atomicOr(&d->flags, ZG_FLAG_SEED_RANGE);
            atomicOr(&d->step_flags, ZG_FLAG_SEED_RANGE);
            v = -1;
        } else {
            const uint32_t bit = 1u << (v & 31);
            if (atomicOr(&s_seen[(uint32_t)v >> 5], bit) & bit) {
                atomicOr(&d->flags, ZG_FLAG_SEED_DUP);
                atomicOr(&d->step_flags, ZG_FLAG_SEED_DUP);
            }
            a.local_id[v] = (int32_t)i;
        }
        a.S[i] = v;
    }
    uint32_t n = a.batch;
    for (int h = 0; h < a.num_hops; ++h) {
        a.launch = h;
        a.fanout = (int32_t)s.fanout[h];
        a.rows_per_wave = 64u / s.fanout[h];
        a.inv_fanout = 65536u / s.fanout[h] + 1u;
        int32_t *const row_ptr = s.row_ptr[h], *const nbr = s.nbr[h];
        uint8_t *const own = h == a.num_hops - 1 ? a.own : nullptr;
        const uint32_t rpw = a.rows_per_wave, step = rpw * (uint32_t)(kHopBlock / 64), stage_rows = a.stage_edges / s.fanout[h];
        uint32_t ebase = 0;
        for (uint32_t c0 = 0; c0 < n; c0 += kHopRows) {
            const uint32_t nrows = n - c0 < (uint32_t)kHopRows ? n - c0 : (uint32_t)kHopRows;
            __syncthreads(); // S is written, the last batch's rows have been read
            if (tid < nrows) sh.v[tid] = a.S[c0 + tid];
            const uint32_t k = load_rows<OffT>(a, sh, nrows, (int)tid), kincl = wave_incl_scan(k);
            if (lane == 63u) sh.wk[wave] = kincl;
            __syncthreads();
            const uint32_t wk = lane < (uint32_t)kHopBlock / 64u ? sh.wk[lane] : 0u, wks = wave_incl_scan(wk);
            const uint32_t batch_edges = lane_value(wks, 63u);
            if (tid < nrows) {
                const uint32_t rp = lane_value(wks, wave) - lane_value(wk, wave) + kincl - k;
                sh.rp[tid] = rp;
                row_ptr[c0 + tid] = (int32_t)(ebase + rp);
            }
            if (tid == 0) sh.rp[nrows] = batch_edges;
            __syncthreads();
            for (uint32_t b0 = 0; b0 < nrows; b0 += stage_rows) {
                const uint32_t b1 = b0 + stage_rows < nrows ? b0 + stage_rows : nrows, e0 = sh.rp[b0], e1 = sh.rp[b1];
                const IdOut last = load_ids(a, sh, key_lo, key_hi, b0 + wave * rpw, b1, step, (int)lane, e0, s_ids);
                if (last.out) s_ids[last.at] = last.id;
                __syncthreads();
                for (uint32_t e = e0 + tid; e < e1; e += (uint32_t)kHopBlock) {
                    const uint32_t edge = ebase + e;
                    if (edge < s.edge_cap[h]) {
                        const int32_t g = s_ids[e - e0];
                        nbr[edge] = g;
                        bool mine = false; // the hop's first edge to reach the vertex: see mark_bit
                        if ((uint32_t)g < a.num_nodes) {
                            const uint32_t bit = 1u << (g & 31);
                            mine = (atomicOr(&s_marks[(uint32_t)g >> 5], bit) & bit) == 0u;
                        }
                        if (own) own[edge] = mine ? 1 : 0;
                    }
                }
                if (b1 < nrows) __syncthreads(); // the ids are reused
            }
            ebase += batch_edges;
        }
        __syncthreads();
        // rank the hop's new vertices, in ascending id behind D_h
        uint4 x[R];
        uint32_t lex[R];
        const uint32_t np = s.words / 4u, room = s.cap[h + 1] - n;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint32_t q = u * (uint32_t)kHopBlock + tid;
            x[u] = make_uint4(0u, 0u, 0u, 0u);
            if (q < np) {
                x[u] = reinterpret_cast<const uint4 *>(s_marks)[q];
                if (piece_any(x[u])) {
                    const uint4 sn = reinterpret_cast<const uint4 *>(s_seen)[q];
                    reinterpret_cast<uint4 *>(s_marks)[q] = make_uint4(0u, 0u, 0u, 0u);
                    x[u].x &= ~sn.x, x[u].y &= ~sn.y, x[u].z &= ~sn.z, x[u].w &= ~sn.w;
                }
            }
        }
        const uint32_t m = rank_pieces<kHopBlock, R>(x, lex, sh.wsum, np, wave, lane);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            uint32_t j = lex[u];
            const uint32_t w0 = (u * (uint32_t)kHopBlock + tid) * 4u;
            if (piece_any(x[u]))
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c) {
                    const uint32_t w = piece_word(x[u], c);
                    if (w) s_seen[w0 + c] |= j < room ? lowest_set_bits(w, room - j) : 0u; // (vertices beyond the cap are dropped)
                    for (uint32_t y = w; y; y &= y - 1u, ++j) {
                        const int32_t gid = (int32_t)(((w0 + c) << 5) + (uint32_t)__ffs((int)y) - 1u);
                        if (j < room) a.S[n + j] = gid;
                        a.local_id[gid] = j < room ? (int32_t)(n + j) : -1;
                    }
                }
        }
        const uint32_t exact = n + m, next = m < room ? exact : s.cap[h + 1];
        if (tid == 0) {
            row_ptr[n] = (int32_t)ebase;
            d->E[h] = ebase;
            d->n_exact[h + 1] = exact;
            d->n[h + 1] = next;
            if (m > room) {
                atomicOr(&d->flags, ZG_FLAG_HOP_OVERFLOW(h));
                atomicOr(&d->step_flags, ZG_FLAG_HOP_OVERFLOW(h));
            }
        }
        n = next;
        __syncthreads(); // ranks and ids are there for the relabel, the marks for the next hop
        if (h < a.num_hops - 1)
            for (uint32_t e = tid; e < ebase && e < s.edge_cap[h]; e += (uint32_t)kHopBlock) {
                const int32_t g = nbr[e];
                s.col[h][e] = (uint32_t)g < a.num_nodes ? a.local_id[g] : -1;
            }
    }
}

struct CloseRoles { // the closing launch's other workgroups
    RelabelArgs rel; // the edges of hop H-2
    RowArgs gat;     // the copy of the frontier's feature rows (their ids are final by now), if the step has no gather launch
};

// The closing launch: ranks the last hop's vertices, half a compute unit's lanes less per ticket than a sampling launch, tickets
// first in the grid: chains of dependent accesses, they all start at once and leave most of the chip to the copy, which is
// bound by bandwidth and runs beside them.  Measured at 110 M vertices, 433 k new ones and a copy of 157 k rows of 512 bytes
// (160 MB, 34 us alone): 54 us; 1024 lanes per ticket, tickets and copy alternating in the grid: 56 us.  Without a copy,
// 2.4 M vertices and 662 k new ones: 18.1 us (21.0 with a word's vertices one after another in a lane and one window of tickets per look:
// the last lane had its up to 28 written 3.3 us after the tile was ranked, and the last tile its prefix 6 us after the last total was out); 72 k
// new, with a copy of 28 MB: 11.2 us (12.8); 142 k new, with a copy of 48 MB: 20 us, with 1024 lanes 26 us.  A byte-marked tile of 8192 words needs 49 KB of LDS with batches
// of 4096 vertices, which leaves a compute unit room for three such workgroups, not four as with 1024: faster all the same, 66.2 -> 60.0 us (40 M
// vertices, 2 M edges in the last hop, a copy of 64 floats a row) and 125.7 -> 124.9 (100 M, 6 M edges, 32 floats).
template <bool BYTES>
__global__ __launch_bounds__(kCloseBlock, 8) void k_close(HopArgs a, CloseRoles o)
{
    constexpr int R = kHopMaxTileWords / 4 / kCloseBlock;
    constexpr uint32_t kBatch = kCloseBatch; // vertices expanded at a time
    __shared__ uint32_t s_drawn, s_base, s_wsum[64];
    extern __shared__ __align__(16) uint32_t s_dyn[]; // see close_lds
    int32_t *const s_v = reinterpret_cast<int32_t *>(s_dyn);
    if (gate_closed(a.gate)) return;
    if (blockIdx.x >= a.blocks) {
        uint32_t b = blockIdx.x - a.blocks;
        if (b < o.rel.blocks) {
            relabel_block(o.rel, b);
            return;
        }
        b -= o.rel.blocks;
        if (BYTES && a.tag.shift != 0 && a.tag.reaches(*o.gat.n_rows)) {
            if (o.gat.vec4)
                gather_unreached_block<4>(o.gat, b, reinterpret_cast<uint8_t *>(a.marks_prev), a.local_id, a.tag, s_v);
            else
                gather_unreached_block<1>(o.gat, b, reinterpret_cast<uint8_t *>(a.marks_prev), a.local_id, a.tag, s_v);
        } else if (o.gat.vec4) {
            gather_rows_block<4>(o.gat, b, s_v);
        } else {
            gather_rows_block<1>(o.gat, b, s_v);
        }
        return;
    }
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    Drmb *d = a.drmb;
    const uint32_t n_old = d->n[a.launch - 1];
    uint32_t tile = blockIdx.x;
    if (a.draw) {
        if (tid == 0) s_drawn = atomicAdd(&d->ticket[a.launch], 1u);
        __syncthreads();
        tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_drawn);
    }
    const size_t tile0 = (size_t)tile * a.words_per_tile;
    const bool tagged = BYTES && a.tag.shift != 0, reach = tagged && a.tag.reaches(n_old);
    uint8_t *const bytes = reinterpret_cast<uint8_t *>(a.marks_prev);
    uint32_t m, rank0 = 0, room = 0;
    const bool by_words = a.words_per_tile <= (uint32_t)kCloseBlock;
    auto take_prefix = [&]() { // the new vertices before this tile
        if (wave == 0u) {
            auto missing = [&](uint32_t t) { return missing_vertices<BYTES>(a, t, lane); };
            const uint32_t c = by_words ? chain_prefix<4>(a.status_cnt, tile, m, d, (int)lane, a.patience, missing)
                                        : chain_prefix<1>(a.status_cnt, tile, m, d, (int)lane, a.patience, missing);
            if (lane == 0) s_base = c;
        }
    };
    auto use_prefix = [&]() {
        rank0 = n_old + (uint32_t)__builtin_amdgcn_readfirstlane((int)s_base);
        room = rank0 < a.cap_rows ? a.cap_rows - rank0 : 0u;
    };
    auto write_out = [&](int32_t gid, uint32_t j, uint32_t mark) { // the tile's new vertex number j
        if (j < room) a.S[rank0 + j] = gid;
        a.local_id[gid] = j < room ? a.tag.entry(rank0 + j, mark) : -1;
    };
    if (by_words) {
        const uint32_t words = a.words_per_tile;
        uint32_t *const s_words = s_dyn + kBatch;
        uint2 *const s_rank = reinterpret_cast<uint2 *>(s_words + words); // a word's new vertices, and those before them
        const TileWord word = load_words<kCloseBlock, BYTES>(a, tile0, words, tid, s_words);
        uint32_t chunk, before;
        m = rank_chunks<kCloseBlock>(word.fresh, a.chunk_log2, words, s_words, s_wsum, tid, chunk, before);
        if (tid == 0) chain_publish(a.status_cnt, tile, m);
        // a whole word is too long a walk for a lane: a vertex per lane
        const bool by_vertex = a.chunk_log2 == 5u;
        if (by_vertex) {
            if (tid < words) s_rank[tid] = make_uint2(chunk, before);
            __syncthreads();
        }
        const uint32_t first = (uint32_t)tile0 << 5;
        for (uint32_t c0 = 0; c0 == 0 || c0 < m; c0 += kBatch) {
            if (c0) __syncthreads(); // the last batch has been read
            if (by_vertex) {
#pragma unroll 4
                for (uint32_t i = tid; i < 32u * words; i += (uint32_t)kCloseBlock) {
                    const uint2 x = s_rank[i >> 5];
                    const uint32_t j = x.y + __popc(x.x & ((1u << (i & 31u)) - 1u)) - c0;
                    if (((x.x >> (i & 31u)) & 1u) && j < kBatch) s_v[j] = (int32_t)(first + i);
                }
            } else {
                expand_chunk(chunk, before, first + (tid << a.chunk_log2), c0, kBatch, s_v);
            }
            if (c0 == 0) take_prefix();
            __syncthreads();
            use_prefix();
#pragma unroll 2
            for (uint32_t i = tid; i < kBatch && c0 + i < m; i += kCloseBlock) {
                const int32_t gid = s_v[i];
                uint32_t mark = 0u;
                if (tagged) {
                    mark = bytes[gid];
                    bytes[gid] = 0;
                }
                write_out(gid, c0 + i, mark);
            }
        }
        if (!reach && tid < words && word.marked) clear_marks<BYTES>(a, tile0 + tid, word, tagged);
    } else {
        uint32_t *const s_words = s_dyn + kBatch;
        const uint32_t np = a.words_per_tile / 4u;
        uint4 x[R];
        uint32_t lex[R];
        load_tile<kCloseBlock, R, BYTES, false>(a, tile0, np, tid, x, s_words, reach);
        m = rank_pieces<kCloseBlock, R>(x, lex, s_wsum, np, wave, lane);
        if (tid == 0) chain_publish(a.status_cnt, tile, m);
        for (uint32_t c0 = 0; c0 == 0 || c0 < m; c0 += kBatch) {
            if (c0) __syncthreads(); // the last batch has been read
            const uint32_t t = own_vector(tid);
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (u * (uint32_t)kCloseBlock + t < np) expand_piece(x[u], lex[u], (uint32_t)tile0 + (u * (uint32_t)kCloseBlock + t) * 4u, c0, kBatch, s_v);
            if (c0 == 0) take_prefix();
            __syncthreads();
            use_prefix();
#pragma unroll 2
            for (uint32_t i = tid; i < kBatch && c0 + i < m; i += kCloseBlock) {
                const int32_t gid = s_v[i];
                uint32_t mark = 0u;
                if (tagged) {
                    mark = bytes[gid];
                    bytes[gid] = 0;
                }
                write_out(gid, c0 + i, mark);
            }
        }
    }
    if (tid == 0 && tile == a.rank_tiles - 1u) { // the last ticket publishes the hop's size
        const int32_t launch = own_scalar(a.launch);
        const uint64_t exact = (uint64_t)rank0 + m;
        d->n_exact[launch] = (uint32_t)exact;
        d->n[launch] = exact < a.cap_rows ? (uint32_t)exact : a.cap_rows;
        if (exact > a.cap_rows) {
            atomicOr(&d->flags, ZG_FLAG_HOP_OVERFLOW(launch - 1));
            atomicOr(&d->step_flags, ZG_FLAG_HOP_OVERFLOW(launch - 1));
        }
    }
}

struct FinishArgs {
    Drmb *drmb;
    const Drmb *gate;       // gated twin: the plan whose step this launch ends
    Mailbox *gate_mailbox;  // ... and its mailbox: the step counts as completed only now
    int32_t defer_completed; // plan with a gated twin behind it: leave `completed` to the twin's last launch
    int32_t enqueued;        // by the host, as a step of the plan: counts as answered
    Mailbox *mailbox;
    const int32_t *S;
    uint32_t *seen;
    uint32_t *log;
    uint64_t *status;       // the chained scans' status words of every launch: back to zero for the next step
    uint64_t status_words;
    int32_t num_hops;
    uint32_t prefetch; // the launch's workgroup that looks for the next step's inputs
    uint32_t blocks;   // workgroups given to this role (0: role absent)
};

// End of step: the "seen" words of this step's frontier vertices (everything in D_{H-1}: the seeds and
// what hops 0..H-2 added) go back to zero - the bitmaps over |V| are never cleared as a whole -, the scan
// state (status words, tile tickets) restarts for the next step, and the step is appended to the device-side
// log; the step counter advances.
// last launch of a step that carries a gated twin: the owner's step is complete whether or not the twin ran
__device__ __forceinline__ void publish_gate_owner(const FinishArgs &a)
{
    __hip_atomic_store(&a.gate_mailbox->answered, a.gate->answered, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&a.gate_mailbox->completed, a.gate->epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One lane of the step's last launch: if the host has already handed over the next step, its mailbox slot is
// copied into the metadata buffer, so that the next step, if it takes its inputs from there, starts without a read of host memory.  Counted from `step`, not from
// `epoch`: a finish workgroup of the same launch advances that one, before or after this lane looks.
__device__ __forceinline__ void prefetch_step_inputs(Drmb *d, const Mailbox *mailbox)
{
    const uint32_t next = d->step + 1u;
    const uint32_t issued = __hip_atomic_load(&mailbox->issued, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
    if ((int32_t)(issued - (next + 1u)) >= 0) {
        const uint32_t slot = next % kMailboxSlots;
        d->pre_seeds = __hip_atomic_load(&mailbox->slot[slot].seeds, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        d->pre_key = __hip_atomic_load(&mailbox->slot[slot].key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        d->pre_epoch = next;
        d->pre_valid = 1u;
    } else {
        d->pre_valid = 0u;
    }
}

__device__ __forceinline__ void finish_block(const FinishArgs &a, uint32_t block)
{
    const uint32_t n = a.drmb->n[a.num_hops - 1];
    const uint32_t i = block * kBlock + threadIdx.x;
    if (i < n) {
        const int32_t g = a.S[i];
        if (g >= 0) a.seen[(uint32_t)g >> 5] = 0u;
    }
    for (uint64_t w = i; w < a.status_words; w += (uint64_t)a.blocks * kBlock) a.status[w] = 0ull;
    if (i == 0) {
        Drmb *d = a.drmb;
        uint32_t drawn = 0u;
        for (int l = 0; l <= a.num_hops; ++l) drawn += d->ticket[l];
        for (int l = 0; l <= a.num_hops; ++l) d->ticket[l] = 0u;
        const uint32_t epoch = d->epoch, answered = d->answered + (uint32_t)a.enqueued;
        d->answered = answered;
        uint32_t *rec = a.log + (size_t)(epoch % kLogCapacity) * ZG_LOG_STRIDE;
        int p = 0;
        rec[p++] = epoch;
        rec[p++] = d->step_flags;
        for (int h = 0; h <= a.num_hops; ++h) rec[p++] = d->n[h];
        for (int h = 0; h < a.num_hops; ++h) rec[p++] = d->E[h];
        for (int h = 1; h <= a.num_hops; ++h) rec[p++] = d->n_exact[h];
        rec[ZG_LOG_STRIDE - 1] = drawn;
        d->epoch = epoch + 1;
        const uint32_t step_flags = d->step_flags;
        d->last_flags = step_flags;
        d->step_flags = 0; // for the next step: its first kernel raises seed bits from many lanes, so nobody resets there
        d->active = (step_flags & kHopOverflowMask) != 0u && a.defer_completed ? 1u : 0u;
        __hip_atomic_store(&a.mailbox->status[epoch % kMailboxSlots], step_flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (!a.defer_completed) {
            __hip_atomic_store(&a.mailbox->answered, answered, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&a.mailbox->completed, epoch + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (a.gate) publish_gate_owner(a);
    }
}

// "Mean-aggregate": out[i,:] = (1/k_i) * sum over row i of in[col[e],:].  A workgroup owns `rows` output
// rows; their row_ptr slice and input-row indices are staged in LDS, then each lane owns one (row, 16-byte
// column piece) pair at a time and accumulates over the row's edges in fp32, in edge order.
// Inside a step the input rows are read from the feature table (addressed by the sampled global ids: feat[nbr_gid[e]]
// is what X[col[e]] holds) and the rows of X that belong to the last hop's newly discovered vertices are written here,
// by the edge that claimed the vertex: the row passes through the registers once instead of being copied by the
// gather and read back from X (at one reference per row, a third less memory traffic for gather + aggregation).
// the lanes' loop of the aggregation: one (row, 16-byte column piece) pair at a time.  ONE_PASS: the input rows come from
// the feature table and the edge that claimed a newly discovered vertex copies the piece into X on the way.  NT: X is
// stored past the caches (nothing reads it again within the step); the table's rows are loaded through them, so that a
// row several edges share comes from memory once
template <int VEC, bool ONE_PASS, bool NT>
__device__ __forceinline__ void aggregate_rows(const RowArgs &a, uint32_t row0, uint32_t rows, int32_t e_begin, uint32_t e_count,
                                               const int32_t *s_rp, const int32_t *s_col, const int32_t *s_dst)
{
    typedef typename VecOf<VEC>::type T;
    const uint32_t total = rows * a.dimv;
    for (uint32_t e = threadIdx.x; e < total; e += kBlock) {
        const uint32_t r = (uint32_t)(((uint64_t)e * a.inv) >> 32);
        const uint32_t piece = (e - r * a.dimv) * VEC, c = piece < a.last ? piece : a.last; // the piece's first element
        const uint32_t b = (uint32_t)(s_rp[r] - e_begin);
        uint32_t k = (uint32_t)(s_rp[r + 1] - s_rp[r]);
        if (b + k > e_count) k = b < e_count ? e_count - b : 0;
        T acc = VecOf<VEC>::zero();
        // eight of the row's edges at a time: all their loads are in flight before the first is added (in edge order)
        for (uint32_t j0 = 0; j0 < k; j0 += 8) {
            int32_t cj[8];
            T v[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) cj[u] = j0 + u < k ? s_col[b + j0 + u] : -1;
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) {
                v[u] = VecOf<VEC>::zero();
                if (cj[u] >= 0) {
                    const T *src = reinterpret_cast<const T *>(a.src + (int64_t)cj[u] * a.ld_src + c);
                    v[u] = *src;
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u)
                if (cj[u] >= 0) {
                    acc += v[u];
                    if (ONE_PASS) { // the hop's first edge to a new vertex copies the piece into X on the way
                        const int32_t dj = s_dst[b + j0 + u];
                        if (dj >= 0) {
                            T *xd = reinterpret_cast<T *>(a.x_dst + (int64_t)dj * a.ld_x + c);
                            if (NT)
                                __builtin_nontemporal_store(v[u], xd);
                            else
                                *xd = v[u];
                        }
                    }
                }
        }
        const T res = k > 0 ? acc / (float)k : VecOf<VEC>::zero();
        T *out = reinterpret_cast<T *>(a.dst + (int64_t)(row0 + r) * a.ld_dst + c);
        if (NT) // (the step does not read the means again either)
            __builtin_nontemporal_store(res, out);
        else
            *out = res;
    }
}

template <int VEC>
__device__ __forceinline__ void aggregate_block(const RowArgs &a, uint32_t block, int32_t *s_mem)
{
    int32_t *s_rp = s_mem;               // [rows+1]
    int32_t *s_col = s_mem + a.rows + 1; // [rows * max_fanout]
    int32_t *s_dst = s_col + a.rows * a.max_fanout; // [rows * max_fanout] when X is written on the way: row of X, or -1
    const uint32_t n = *a.n_rows;
    const uint32_t n_ids = *a.n_cols, n_in = a.col_out ? a.col_limit : n_ids;
    const int32_t x_from = !a.own && a.tag.shift != 0 && a.tag.reaches(n) ? 0 : (int32_t)n;
    const uint32_t row0 = block * a.rows;
    if (row0 >= n) return;
    const uint32_t rows = n - row0 < a.rows ? n - row0 : a.rows;
    for (uint32_t t = threadIdx.x; t <= rows; t += kBlock) s_rp[t] = a.row_ptr[row0 + t];
    __syncthreads();
    const int32_t e_begin = s_rp[0];
    uint32_t e_count = (uint32_t)(s_rp[rows] - e_begin);
    if (e_count > a.rows * a.max_fanout) e_count = a.rows * a.max_fanout;
    for (uint32_t t = threadIdx.x; t < e_count; t += kBlock) { // input row of every edge, -1 = none
        const uint32_t c = (uint32_t)a.col[e_begin + t];
        const bool valid = c < n_in;
        s_col[t] = valid ? (int32_t)c : -1;
        if (a.col_out) { // "relabel edges" of this block, done here: c is the sampled global id
            const int32_t entry = valid ? a.local_id[c] : -1;
            const int32_t id = a.tag.local_id(entry), lid = (uint32_t)id < n_ids ? id : -1;
            a.col_out[e_begin + t] = lid;
            // one edge to a vertex writes its row of X, if the vertex is new or the frontier's rows are not the copy's
            if (a.x_dst) s_dst[t] = lid >= x_from && (a.own ? a.own[e_begin + t] != 0 : a.tag.owns(entry, (uint32_t)(e_begin + (int32_t)t))) ? lid : -1;
        }
    }
    __syncthreads();
    if (a.x_dst)
        aggregate_rows<VEC, true, true>(a, row0, rows, e_begin, e_count, s_rp, s_col, s_dst);
    else if (a.nt)
        aggregate_rows<VEC, false, true>(a, row0, rows, e_begin, e_count, s_rp, s_col, s_dst);
    else
        aggregate_rows<VEC, false, false>(a, row0, rows, e_begin, e_count, s_rp, s_col, s_dst);
}

// The two bandwidth-bound launches of a step, each with a small companion role on its last workgroups:
// {gather + relabel of the last hop}, then {aggregation + end-of-step clean-up}.  An absent role has zero
// workgroups (the stand-alone entry points launch the big role alone).
template <int VEC>
__global__ __launch_bounds__(kBlock) void k_gather(RowArgs gat, RelabelArgs last)
{
    extern __shared__ int32_t s_mem[];
    if (gate_closed(last.gate)) return;
    // the relabel's workgroups come first: their chains of dependent loads then run under the copy instead of after it
    if (blockIdx.x < last.blocks)
        relabel_block(last, blockIdx.x);
    else
        gather_block<VEC>(gat, blockIdx.x - last.blocks, s_mem);
}

// (a small step has no closing launch to copy the frontier's rows in: they come first here)
struct NoCopy {};
__device__ __forceinline__ uint32_t copy_blocks(const RowArgs &copy) { return copy.blocks; }
__device__ __forceinline__ uint32_t copy_blocks(const NoCopy &) { return 0u; }
template <int VEC> __device__ __forceinline__ void copy_block(const RowArgs &copy, uint32_t b, int32_t *s_id) { gather_rows_block<VEC>(copy, b, s_id); }
template <int VEC> __device__ __forceinline__ void copy_block(const NoCopy &, uint32_t, int32_t *) {}

template <int VEC, class Copy>
__global__ __launch_bounds__(kBlock) void k_aggregate(RowArgs agg, FinishArgs fin, Copy copy)
{
    extern __shared__ int32_t s_mem[];
    if (gate_closed(fin.gate)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) publish_gate_owner(fin);
        return;
    }
    if (blockIdx.x == fin.prefetch && threadIdx.x == 0 && fin.blocks && !fin.gate) prefetch_step_inputs(fin.drmb, fin.mailbox);
    const uint32_t copies = copy_blocks(copy);
    if (blockIdx.x < copies)
        copy_block<VEC>(copy, blockIdx.x, s_mem);
    else if (blockIdx.x - copies < agg.blocks)
        aggregate_block<VEC>(agg, blockIdx.x - copies, s_mem);
    else
        finish_block(fin, blockIdx.x - copies - agg.blocks);
}

// The tail of a step without features: relabel of the last hop and end-of-step clean-up, in one launch - neither reads what the
// other writes (two launches: 21 + 6 us and a boundary at 2 M edges).
__global__ __launch_bounds__(kBlock) void k_tail(RelabelArgs last, FinishArgs fin)
{
    if (gate_closed(fin.gate)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) publish_gate_owner(fin);
        return;
    }
    if (blockIdx.x == fin.prefetch && threadIdx.x == 0 && !fin.gate) prefetch_step_inputs(fin.drmb, fin.mailbox);
    if (blockIdx.x < last.blocks)
        relabel_block(last, blockIdx.x);
    else
        finish_block(fin, blockIdx.x - last.blocks);
}

// plain streaming copy of 16-byte pieces: the traffic counters' calibration kernel (zg_calibration_copy)
__global__ __launch_bounds__(kBlock) void k_calibrate_copy(const uint4 *src, uint4 *dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) dst[i] = src[i];
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// graph check: indices in range and rows strictly ascending
template <typename OffT>
__global__ void k_validate(const OffT *off, const int32_t *idx, int64_t num_nodes, uint32_t *bad)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < num_nodes; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = (int64_t)off[v], e = (int64_t)off[v + 1];
        int32_t prev = -1;
        for (int64_t p = b; p < e; ++p) {
            const int32_t g = idx[p];
            if (g < 0 || (int64_t)g >= num_nodes) atomicOr(bad, 1u);
            if (g <= prev) atomicOr(bad, 2u);
            prev = g;
        }
    }
}

// ---- graph-aware size model (plan time) ---------------------------------------------------------
// The size model of the paper's Lemma 1 treats every neighbor draw as an independent pick of a vertex with
// probability proportional to its degree.  The kernels below keep its frame - the size of D_h is a sum of
// independent indicators, one per vertex - but take each vertex's inclusion probability from the graph itself:
// with q_u = P(u in D_h) and r_u = the chance that a given neighbor of u is among u's picks at hop h
// (min(F, deg)/deg without replacement, 1 - (1 - 1/deg)^F with), a vertex v stays out of D_{h+1} with
// probability (1 - q_v) * prod over its in-neighbors u of (1 - q_u r_u).  One sweep over the edges per hop.
// Sums are kept as 64-bit fixed point (2^-32) so that the result does not depend on the order of the atomics.
constexpr double kFix = 4294967296.0; // 2^32
constexpr int kModelBinBlock = 512, kModelWindow = 4096; // threads of a workgroup of k_model_bin, edges it looks at together
constexpr int kModelAddBlock(bool terms) { return terms ? 512 : 1024; }
constexpr uint32_t kModelMaxBins = 32768;                // a counter each in LDS
constexpr uint32_t kModelSlices = 8;                     // one per XCD
constexpr uint32_t kModelNoShare = 0xFFFFFFFFu;
constexpr int64_t kModelMinPart = 16384;
constexpr int64_t kModelRowsNodes = 1 << 19;             // rows whose terms an XCD's L2 holds
constexpr int kModelBlock = 1024, kModelGrid = 512; // the sweeps over the vertices
constexpr int64_t kModelPushWaves = 16384;          // twice what the chip holds at once
constexpr int64_t kModelRowWork = 1;                // a row of a sweep by atomics, in edges

// What a sweep by atomics has to do for a vertex that may be in D_h, in edges: the graph's offsets, where that is summed up
struct ModelRows {
    const void *off;
    int32_t wide;
    __device__ __forceinline__ unsigned long long work(int64_t v) const
    {
        const int64_t deg = wide ? ((const int64_t *)off)[v + 1] - ((const int64_t *)off)[v] : (int64_t)(((const int32_t *)off)[v + 1] - ((const int32_t *)off)[v]);
        return deg > 0 ? (unsigned long long)(deg + kModelRowWork) : 0ull;
    }
};

// ... and what depends on the sum: a kernel of the first hop that may not be meant to run (see zg_envelope_model_graph)
struct ModelGate {
    const unsigned long long *work; // null: always
    unsigned long long below;
    __device__ __forceinline__ bool closed() const { return work != nullptr && *work >= below; }
};

// the workgroup's sums of x[0 .. N-1] into out[0 .. N-1] (all lanes; one instruction: atomics queue up at 13 ns)
template <int NT, int N>
__device__ __forceinline__ void add_sums(unsigned long long *out, unsigned long long (&x)[N])
{
    __shared__ unsigned long long s_sum[N][NT / 64];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] += __shfl_xor(x[i], d, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) s_sum[i][threadIdx.x >> 6] = x[i];
    __syncthreads();
    if (threadIdx.x < N) {
        unsigned long long sum = 0ull;
        for (int w = 0; w < NT / 64; ++w) sum += s_sum[threadIdx.x][w];
        atomicAdd(&out[threadIdx.x], sum);
    }
}

template <bool COUNT>
__global__ __launch_bounds__(COUNT ? kModelBlock : kBlock) void k_model_init(float *q, unsigned long long *ell, const float *seed_prob, float uniform, int64_t n,
                                                                             ModelRows rows, unsigned long long *work)
{
    unsigned long long sum[1] = {0ull};
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        float p = seed_prob ? seed_prob[v] : uniform;
        p = p < 0.0f ? 0.0f : (p > 1.0f ? 1.0f : p);
        q[v] = p;
        ell[v] = 0ull;
        if (COUNT && p > 0.0f) sum[0] += rows.work(v);
    }
    if (COUNT) add_sums<kModelBlock>(work, sum);
}

// -log(1 - q_u r_u) in fixed point: what a vertex u of `deg` neighbors adds to each of them (at most 9e10: 37 bits)
__device__ __forceinline__ unsigned long long model_term(float qu, int64_t deg, int32_t fanout, int32_t replace)
{
    if (qu <= 0.0f || deg <= 0) return 0ull;
    double r;
    if (replace)
        r = -expm1((double)fanout * log1p(-1.0 / (double)deg));
    else
        r = deg <= fanout ? 1.0 : (double)fanout / (double)deg;
    double x = (double)qu * r;
    if (x > 1.0 - 1e-9) x = 1.0 - 1e-9;
    return (unsigned long long)(-log1p(-x) * kFix);
}

// The sweep with nothing but the two arrays over the vertices: one 64-bit atomic per edge that has a term, a wave per source
// vertex.  Bound by the atomics: 16 G/s here, whatever their scope - the L2s pass every one on to memory (7 ms per hop at 120 M edges).
// Where few vertices can be in D_h the rest have to be passed by quickly: a wave looks at `rows` vertices at a time, a lane each (a power of
// two; as many as leave enough waves).  One vertex at a time took 75 ps each: 2.4 M vertices and 115 M edges, 1 % of the vertices as
// seeds, 213 -> 106 us for the call.  (Where that is one vertex, the plain loop: 15.5 instead of 16.8 us at 30 k vertices and 2^18 edges.)
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_model_push(const OffT *off, const int32_t *idx, const float *q, unsigned long long *ell,
                                                       int64_t n, int32_t fanout, int32_t replace, int32_t rows, ModelGate gate)
{
    if (gate.closed()) return;
    const int lane = threadIdx.x & 63;
    const int64_t wave0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int64_t waves = ((int64_t)gridDim.x * kBlock) >> 6;
    for (int64_t u = wave0; rows == 1 && u < n; u += waves) {
        const int64_t b = (int64_t)off[u], e = (int64_t)off[u + 1];
        const unsigned long long c = model_term(q[u], e - b, fanout, replace);
        if (c == 0ull) continue;
        for (int64_t p = b + lane; p < e; p += 64) atomicAdd(&ell[idx[p]], c);
    }
    if (rows == 1) return;
    for (int64_t u0 = wave0 * rows; u0 < n; u0 += waves * rows) {
        const int64_t u = u0 + lane;
        float qu = 0.0f;
        int64_t b = 0, e = 0;
        if (lane < rows && u < n) {
            qu = q[u];
            if (rows < 64 || qu > 0.0f) { // (a small graph's offsets are not worth waiting for q)
                b = (int64_t)off[u];
                e = (int64_t)off[u + 1];
            }
        }
        const unsigned long long c = model_term(qu, e - b, fanout, replace);
        for (unsigned long long some = __ballot(c != 0ull); some; some &= some - 1ull) {
            const uint32_t l = (uint32_t)__ffsll((long long)some) - 1u;
            auto of = [&](unsigned long long x) { return (unsigned long long)lane_value((uint32_t)(x >> 32), l) << 32 | lane_value((uint32_t)x, l); };
            const int64_t first = (int64_t)of((unsigned long long)b), end = (int64_t)of((unsigned long long)e);
            const unsigned long long term = of(c);
            for (int64_t p = first + lane; p < end; p += 64) atomicAdd(&ell[idx[p]], term);
        }
    }
}

// The sweep with room for 9 bytes per edge: no atomic leaves a compute unit.  The vertices are cut into bins of 2^log2.  Once per
// call the edges are counted by chunk and bin (k_model_count), the counts turned into places (k_model_places, k_model_starts) and every edge
// written to its neighbor's bin behind those of earlier chunks (k_model_bin): its row's low bits, and the neighbor within the bin.  A chunk's rows
// are all of one block of rows (k_model_chunks), so a bin's entries are runs of one block each, in which the low bits are enough.  In
// each hop the rows' terms are worked out once (k_model_terms); a workgroup per bin, or several, goes through its entries, looks
// their terms up and adds them up in LDS (k_model_add).  The terms are integers: the same sums as above.
// k_model_bin's stores are a line for nearly each edge (115 M: 0.47 ms, 245 G/s), so it runs once and not in every hop, and puts a window's entries in the order of
// their bins in LDS first, from where they leave in runs (0.37 ms); k_model_add is bound by its look-ups, whose lines have to come out of the L2: out of memory they come at 58 G/s (0.58 ms a hop at 2.4 M vertices).  Terms of 2^19 rows
// fit one; up to 2^22 rows, each XCD's workgroups take a slice of them, an eighth, and k_model_update adds the eight slices' sums up (0.28 ms
// and 0.035, with 2.2 entries per look-up's line; bins half as large 0.33).  Beyond, or where the slices' sums do not fit (fewer than 16 edges
// per vertex), an entry holds its term and the neighbor, 8 bytes, and k_model_bin runs in every hop (16 M vertices, 144 M edges, two hops:
// 4.0 ms; by look-ups 6.3).
// Atomics / 8-byte entries in every hop / now, ms: three hops, 2.4 M vertices and 115 M edges 22.8 / 3.29 / 1.61, one hop 1.23 / 0.92; 250 k and 83 M
// 2.45 / 0.94; 100 k and 29 M 0.82 / 0.31; 300 k and 3.5 M 0.26 / 0.20; two hops, 3.9 M and 113 M 2.35 / 1.53; 700 k and 13 M 0.34 / 0.29.
struct ModelBins {
    const int32_t *idx;
    int64_t num_edges, num_nodes;
    uint32_t log2, bins;
    uint32_t block_log2, blocks; // rows of a block, and how many blocks there are
    uint32_t chunk, chunks;      // edges of a chunk at most, a multiple of kModelWindow, and how many chunks there are at most
    uint32_t part, parts;        // most entries a workgroup of k_model_add takes, and how many such parts there are at most
    uint32_t *first_chunk;       // [blocks + 1]: of each block of rows
    uint32_t *chunk_edge;        // [chunks + 1]: where the chunk begins
    uint32_t *place;             // [bins][chunks]: edges of the chunk that lead into the bin; then how many of earlier chunks do
    uint32_t *start;             // [bins + 1]: where the bin's entries begin
    uint32_t *share;             // [parts]: a bin, and above its 15 bits which part of it; kModelNoShare behind the last one
    void *entry;                 // [num_edges]: 4 bytes, or 8 where an entry holds its term
    unsigned long long *term;    // [num_nodes] the rows' terms; null: the entries hold them
    uint32_t slices;             // of the rows' blocks, a workgroup of k_model_add each
    unsigned long long *more;    // [slices - 1][num_nodes]: the sums of the slices behind the first (of bins in one part)
    unsigned long long *sums;    // [2 num_hops]: of all hops
};

// one workgroup: the blocks' first chunks and all chunks' first edges
template <typename OffT>
__global__ __launch_bounds__(1024) void k_model_chunks(ModelBins m, const OffT *off)
{
    extern __shared__ uint32_t s_first[]; // [blocks]
    __shared__ uint32_t s_sum[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, each = (m.blocks + 1023u) / 1024u;
    auto edge_of = [&](uint32_t k) { // block k's first edge
        const int64_t r = (int64_t)k << m.block_log2;
        return (uint32_t)(int64_t)off[r < m.num_nodes ? r : m.num_nodes];
    };
    const uint32_t k0 = tid * each < m.blocks ? tid * each : m.blocks, k1 = k0 + each < m.blocks ? k0 + each : m.blocks;
    uint32_t sum = 0;
    auto chunks_of = [&](uint32_t k) { // (edges + chunk - 1 may be 2^32 or more)
        const uint32_t edges = edge_of(k + 1u) - edge_of(k);
        return edges / m.chunk + (edges % m.chunk != 0u ? 1u : 0u);
    };
    for (uint32_t k = k0; k < k1; ++k) sum += chunks_of(k);
    const uint32_t incl = wave_incl_scan(sum);
    if (lane == 63u) s_sum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum, total = 0;
    for (uint32_t w = 0; w < 16u; ++w) {
        if (w < wave) run += s_sum[w];
        total += s_sum[w];
    }
    for (uint32_t k = k0; k < k1; ++k) {
        s_first[k] = m.first_chunk[k] = run;
        run += chunks_of(k);
    }
    if (tid == 0) m.first_chunk[m.blocks] = total;
    __syncthreads();
    for (uint32_t c = tid; c <= m.chunks; c += 1024u) {
        uint32_t lo = 0, hi = m.blocks; // the last block whose first chunk is not behind c (blocks without edges have none of their own)
        while (hi - lo > 1u) {
            const uint32_t mid = (lo + hi) / 2u;
            if (s_first[mid] <= c)
                lo = mid;
            else
                hi = mid;
        }
        m.chunk_edge[c] = c < total ? edge_of(lo) + (c - s_first[lo]) * m.chunk : (uint32_t)m.num_edges;
    }
}

__global__ __launch_bounds__(1024) void k_model_count(ModelBins m)
{
    extern __shared__ uint32_t s_count[];
    for (uint32_t b = threadIdx.x; b < m.bins; b += 1024u) s_count[b] = 0u;
    __syncthreads();
    const int64_t e0 = m.chunk_edge[blockIdx.x], e1 = m.chunk_edge[blockIdx.x + 1u];
    typedef int32_t v4i __attribute__((ext_vector_type(4), aligned(4)));
    auto count = [&](int32_t id) {
        const uint32_t g = (uint32_t)id;
        if ((int64_t)g < m.num_nodes) atomicAdd(&s_count[g >> m.log2], 1u);
    };
    const int64_t e4 = e0 + (e1 - e0) / 4 * 4;
#pragma unroll 4
    for (int64_t e = e0 + 4 * (int64_t)threadIdx.x; e < e4; e += 4096) {
        const v4i x = *reinterpret_cast<const v4i *>(m.idx + e);
        count(x[0]);
        count(x[1]);
        count(x[2]);
        count(x[3]);
    }
    if (e4 + threadIdx.x < e1) count(m.idx[e4 + threadIdx.x]);
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < m.bins; b += 1024u) m.place[(size_t)b * m.chunks + blockIdx.x] = s_count[b];
}

// a workgroup per bin: the running sums over the chunks; start[b] = the bin's total
__global__ __launch_bounds__(256) void k_model_places(ModelBins m)
{
    __shared__ uint32_t s_sum[4];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    uint32_t *const place = m.place + (size_t)blockIdx.x * m.chunks;
    uint32_t run = 0;
    for (uint32_t c0 = 0; c0 < m.chunks; c0 += 2048u) {
        uint32_t x[8], sum = 0;
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u) {
            const uint32_t c = c0 + tid * 8u + u;
            x[u] = c < m.chunks ? place[c] : 0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u) sum += x[u];
        const uint32_t incl = wave_incl_scan(sum);
        if (lane == 63u) s_sum[wave] = incl;
        __syncthreads();
        uint32_t before = run + incl - sum;
        for (uint32_t w = 0; w < 4u; ++w) {
            if (w < wave) before += s_sum[w];
            run += s_sum[w];
        }
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u) {
            const uint32_t c = c0 + tid * 8u + u;
            if (c < m.chunks) place[c] = before;
            before += x[u];
        }
        __syncthreads();
    }
    if (tid == 0) m.start[blockIdx.x] = run;
}

__device__ __forceinline__ uint32_t model_parts(const ModelBins &m, uint32_t entries) { return entries > m.part ? (entries - 1u) / m.part + 1u : 1u; }

// one workgroup: the bins' totals into their starts, and the bins into parts of at most m.part entries; the hops' sums start at zero
__global__ __launch_bounds__(1024) void k_model_starts(ModelBins m)
{
    __shared__ uint32_t s_sum[2][16];
    if (threadIdx.x < 2u * ZG_MAX_HOPS) m.sums[threadIdx.x] = 0ull;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, each = (m.bins + 1023u) / 1024u;
    const uint32_t b0 = threadIdx.x * each < m.bins ? threadIdx.x * each : m.bins, b1 = b0 + each < m.bins ? b0 + each : m.bins;
    uint32_t sum = 0, parts = 0;
    for (uint32_t b = b0; b < b1; ++b) {
        sum += m.start[b];
        parts += model_parts(m, m.start[b]);
    }
    const uint32_t incl = wave_incl_scan(sum), incl_parts = wave_incl_scan(parts);
    if (lane == 63u) {
        s_sum[0][wave] = incl;
        s_sum[1][wave] = incl_parts;
    }
    __syncthreads();
    uint32_t run = incl - sum, at = incl_parts - parts, end = 0;
    for (uint32_t w = 0; w < 16u; ++w) {
        if (w < wave) run += s_sum[0][w];
        if (w < wave) at += s_sum[1][w];
        end += s_sum[1][w];
    }
    for (uint32_t i = end + threadIdx.x; i < m.parts; i += 1024u) m.share[i] = kModelNoShare;
    for (uint32_t b = b0; b < b1; ++b) {
        const uint32_t x = m.start[b], p = model_parts(m, x);
        m.start[b] = run;
        run += x;
        for (uint32_t i = 0; i < p; ++i) m.share[at++] = b | (i << 15);
    }
    if (threadIdx.x == 1023u) m.start[m.bins] = run; // (threads without bins carry the total on)
}

__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v)
{
    auto up = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = up(v, dpp_or_zero<0x111, 0xF>(v));
    v = up(v, dpp_or_zero<0x112, 0xF>(v));
    v = up(v, dpp_or_zero<0x114, 0xF>(v));
    v = up(v, dpp_or_zero<0x118, 0xF>(v));
    v = up(v, dpp_or_zero<0x142, 0xA>(v));
    v = up(v, dpp_or_zero<0x143, 0xC>(v));
    return v;
}

// A workgroup goes through a chunk of the edges in windows: the rows that begin in the window leave their number at their first
// edge, a running maximum tells every edge its row, and the row - with TERMS its term, worked out once, by a thread per row - goes to the edge's bin.
template <typename OffT, bool TERMS>
__global__ __launch_bounds__(kModelBinBlock, 4) void k_model_bin(ModelBins m, const OffT *off, const float *q, int32_t fanout, int32_t replace)
{
    constexpr uint32_t kEach = kModelWindow / kModelBinBlock, NW = kModelBinBlock / 64;
    typedef int32_t v4i __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ __align__(16) uint16_t s_row[kModelWindow]; // at a row's first edge in the window: the row, counted from the window's first
    __shared__ unsigned long long s_term[TERMS ? kModelBinBlock : 1];
    __shared__ unsigned long long s_last;
    __shared__ uint32_t s_max[NW], s_count[TERMS ? 1 : kModelBinBlock];
    __shared__ uint2 s_first[TERMS ? 1 : kModelBinBlock], s_item[TERMS ? 1 : kModelWindow];
    extern __shared__ uint32_t s_next[]; // where the bin's next entry goes
    if (!TERMS) s_count[threadIdx.x] = 0u;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const int64_t n = m.num_nodes;
    for (uint32_t b = tid; b < m.bins; b += (uint32_t)kModelBinBlock) s_next[b] = m.start[b] + m.place[(size_t)b * m.chunks + blockIdx.x];
    int64_t e = m.chunk_edge[blockIdx.x];
    const int64_t e1 = m.chunk_edge[blockIdx.x + 1u];
    if (e >= e1) return;
    // the row that holds edge e: off[row] <= e < off[row + 1], a thread per probe
    int64_t row = 0, hi = n;
    while (hi - row > 1) {
        const int64_t step = (hi - row + kModelBinBlock - 1) / kModelBinBlock, p = row + ((int64_t)tid + 1) * step;
        row += (int64_t)__syncthreads_count(p < hi && (int64_t)off[p] <= e) * step;
        if (row + step < hi) hi = row + step;
    }
    // this thread's edges, and the rows row .. row + kModelBinBlock - 1, one per thread: loaded a window ahead
    v4i v_next[kEach / 4];
    int64_t o0_next, o1_next;
    float q_next;
    auto load_window = [&]() {
#pragma unroll
        for (uint32_t u = 0; u < kEach / 4; ++u) {
            const int64_t p = e + (int64_t)tid * kEach + 4 * u;
            if (p + 4 <= e1) {
                v_next[u] = *reinterpret_cast<const v4i *>(m.idx + p);
            } else {
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i) v_next[u][i] = p + i < e1 ? m.idx[p + i] : -1;
            }
        }
        const int64_t r = row + tid;
        o0_next = (int64_t)off[r < n ? r : n];
        o1_next = (int64_t)off[r + 1 < n ? r + 1 : n];
        q_next = TERMS && r < n ? q[r] : 0.0f;
    };
    load_window();
    while (e < e1) {
        v4i v[kEach / 4];
#pragma unroll
        for (uint32_t u = 0; u < kEach / 4; ++u) v[u] = v_next[u];
        const int64_t mine = e + (int64_t)tid * kEach, o0 = o0_next, o1 = o1_next, r = row + tid, e_now = e;
        const float qr = q_next;
        if (tid == kModelBinBlock - 1) s_last = (unsigned long long)o1;
#pragma unroll
        for (uint32_t u = 0; u < kEach / 4; ++u) reinterpret_cast<uint2 *>(s_row)[tid * (kEach / 4) + u] = make_uint2(0u, 0u);
        __syncthreads();
        int64_t w1 = e + kModelWindow < e1 ? e + kModelWindow : e1; // the window's end; earlier if it has more rows than there are threads
        if ((int64_t)s_last < w1) w1 = (int64_t)s_last;
        row += __syncthreads_count(r < n && o1 <= w1);
        e = w1;
        if (e < e1) load_window();
        if (o1 > o0 && o1 > e_now && o0 < w1) {
            s_row[o0 > e_now ? o0 - e_now : 0] = (uint16_t)tid;
            if (TERMS) s_term[tid] = model_term(qr, o1 - o0, fanout, replace);
        }
        __syncthreads();
        uint32_t at[kEach], rank[kEach], top = 0;
#pragma unroll
        for (uint32_t u = 0; u < kEach; ++u) {
            const uint32_t x = s_row[tid * kEach + u];
            top = x > top ? x : top;
            at[u] = top;
        }
        const uint32_t incl = wave_incl_max(top);
        uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x138, 0xF, 0xF, true); // (the lane before: wave_shr:1)
        if (lane == 63u) s_max[wave] = incl;
        __syncthreads();
        const uint32_t others = lane_value(wave_incl_max(lane < wave ? s_max[lane] : 0u), 63u);
        before = before > others ? before : others;
#pragma unroll
        for (uint32_t u = 0; u < kEach; ++u) {
            const uint32_t g = (uint32_t)v[u / 4][u % 4];
            const bool there = mine + u < w1 && (int64_t)g < n;
            const uint32_t x = at[u] > before ? at[u] : before, in_bin = g & ((1u << m.log2) - 1u);
            if (TERMS) {
                if (there) static_cast<unsigned long long *>(m.entry)[atomicAdd(&s_next[g >> m.log2], 1u)] = (s_term[x] << m.log2) | in_bin;
            } else { // the row's low bits; the entry's number within the window and its bin
                at[u] = (((uint32_t)(r - tid) + x) << m.log2) | in_bin;
                rank[u] = there ? atomicAdd(&s_count[g >> m.log2], 1u) : 0xFFFFFFFFu;
            }
        }
        if (!TERMS) { // the window's entries in the order of their bins, so that they leave in runs
            __syncthreads();
            const uint32_t c = tid < m.bins ? s_count[tid] : 0u, sum = wave_incl_scan(c);
            if (lane == 63u) s_max[wave] = sum;
            __syncthreads();
            const uint32_t w = lane < NW ? s_max[lane] : 0u, ws = wave_incl_scan(w), first = lane_value(ws, wave) - lane_value(w, wave) + sum - c, total = lane_value(ws, 63u);
            if (tid < m.bins) {
                s_first[tid] = make_uint2(first, s_next[tid]);
                s_next[tid] += c;
                s_count[tid] = 0u;
            }
            __syncthreads();
#pragma unroll
            for (uint32_t u = 0; u < kEach; ++u)
                if (rank[u] != 0xFFFFFFFFu) {
                    const uint2 f = s_first[(uint32_t)v[u / 4][u % 4] >> m.log2];
                    s_item[f.x + rank[u]] = make_uint2(at[u], f.y + rank[u]);
                }
            __syncthreads();
#pragma unroll 2
            for (uint32_t i = tid; i < total; i += (uint32_t)kModelBinBlock) {
                const uint2 y = s_item[i];
                static_cast<uint32_t *>(m.entry)[y.y] = y.x;
            }
        }
    }
}

// A workgroup per bin, or per part of a bin that holds more than twice its share of the edges (hubs, ids in the order of their
// popularity): the parts' sums meet in `ell`, which is zero before.  One workgroup went through such a bin at an entry per clock: three
// hops at 2.4 M vertices and 115 M edges 64.4 ms with ids in the order of a power law's ranks, 147 ms with half of the edges into
// one vertex; in parts 3.1 and 4.1 ms (3.0 with even bins).  Parts of one share cut every bin in two, and with them all sums go through
// atomics (2.4 M more per hop); fewer than 256 bins are cut as if they were 256.
template <bool TERMS>
__global__ __launch_bounds__(kModelAddBlock(TERMS)) void k_model_add(ModelBins m, unsigned long long *ell)
{
    constexpr uint32_t NT = kModelAddBlock(TERMS);
    extern __shared__ unsigned long long s_ell[];
    const uint32_t slice = TERMS ? 0u : blockIdx.x % m.slices, share = m.share[TERMS ? blockIdx.x : blockIdx.x / m.slices];
    if (share == kModelNoShare) return;
    const uint32_t bin = share & (kModelMaxBins - 1u), size = 1u << m.log2, mask = size - 1u;
    const uint32_t b0 = m.start[bin], all = m.start[bin + 1u] - b0, e0 = (share >> 15) * m.part, e1 = all - e0 < m.part ? all : e0 + m.part;
    for (uint32_t i = threadIdx.x; i < size; i += NT) s_ell[i] = 0ull;
    __syncthreads();
    if (TERMS) {
        typedef unsigned long long v2u __attribute__((ext_vector_type(2), aligned(8)));
        const unsigned long long *const entry = static_cast<const unsigned long long *>(m.entry) + b0;
        const uint32_t pairs = (e1 - e0) / 2u;
#pragma unroll 4
        for (uint32_t i = threadIdx.x; i < pairs; i += NT) {
            const v2u x = *reinterpret_cast<const v2u *>(entry + e0 + 2u * (size_t)i);
            atomicAdd(&s_ell[(uint32_t)x[0] & mask], x[0] >> m.log2);
            atomicAdd(&s_ell[(uint32_t)x[1] & mask], x[1] >> m.log2);
        }
        if (threadIdx.x == 0 && ((e1 - e0) & 1u)) {
            const unsigned long long x = entry[e1 - 1u];
            atomicAdd(&s_ell[(uint32_t)x & mask], x >> m.log2);
        }
    } else {
        constexpr uint32_t U = 8; // entries of a lane, and then their terms, on the way at once
        const uint32_t *const entry = static_cast<const uint32_t *>(m.entry) + b0, *const place = m.place + (size_t)bin * m.chunks;
        auto run_of = [&](uint32_t k) { // the bin's first entry of block k
            const uint32_t c = m.first_chunk[k];
            return c < m.chunks ? place[c] : all;
        };
        const uint32_t k0 = m.blocks * slice / m.slices, k1 = m.blocks * (slice + 1u) / m.slices;
        uint32_t next = run_of(k0);
        for (uint32_t k = k0; k < k1 && next < e1; ++k) {
            const uint32_t r0 = next > e0 ? next : e0;
            next = run_of(k + 1u);
            const uint32_t r1 = next < e1 ? next : e1;
            const unsigned long long *const term = m.term + ((size_t)k << m.block_log2);
            const uint32_t in_block = (1u << m.block_log2) - 1u;
            const uint32_t *const run = entry + r0;
            const uint32_t count = r1 > r0 ? r1 - r0 : 0u; // at most m.part, 2^25: the sums below stay within 32 bits, which r1 may fill
            for (uint32_t i = threadIdx.x; i < count; i += U * NT) {
                uint32_t x[U];
                unsigned long long t[U];
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) x[u] = i + u * NT < count ? run[i + u * NT] : 0xFFFFFFFFu;
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) t[u] = i + u * NT < count ? term[(x[u] >> m.log2) & in_block] : 0ull;
#pragma unroll
                for (uint32_t u = 0; u < U; ++u)
                    if (t[u]) atomicAdd(&s_ell[x[u] & mask], t[u]);
            }
        }
    }
    __syncthreads();
    const int64_t v0 = (int64_t)bin << m.log2;
    const bool alone = all <= m.part;
    for (uint32_t i = threadIdx.x; i < size && v0 + i < m.num_nodes; i += NT) {
        const unsigned long long x = s_ell[i];
        if (alone)
            (slice ? m.more + (size_t)(slice - 1u) * m.num_nodes : ell)[v0 + i] = x;
        else if (x)
            atomicAdd(&ell[v0 + i], x);
    }
}

// the rows' terms of a hop
template <typename OffT>
__global__ __launch_bounds__(kBlock) void k_model_terms(const OffT *off, const float *q, unsigned long long *term, int64_t n, int32_t fanout, int32_t replace)
{
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (v < n) term[v] = model_term(q[v], (int64_t)off[v + 1] - (int64_t)off[v], fanout, replace);
}

// q_v <- 1 - (1 - q_v) exp(-ell_v); ell_v <- 0; sums[0] += q_v, sums[1] += q_v (1 - q_v); with COUNT, sums[2] += the next sweep's
// work.  Vertices kModelStride apart are added in double, everything else as integers, so the sums do not depend on the launch.  One pair of atomics per workgroup of at most
// 512: a pair per wavefront queued up on the two words (2.4 M vertices: 905 us, now 16 us).
constexpr int64_t kModelStride = (int64_t)65536 * kBlock;
struct ModelSlices { // what k_model_add left beside `ell`
    const unsigned long long *more;
    uint32_t count; // arrays of it
    const uint32_t *start;
    uint32_t log2, part;
};

template <bool COUNT>
__global__ __launch_bounds__(kModelBlock) void k_model_update(float *q, unsigned long long *ell, int64_t n, unsigned long long *sums, ModelGate gate,
                                                              ModelRows rows, ModelSlices slices)
{
    if (gate.closed()) return;
    unsigned long long sum[COUNT ? 3 : 2] = {};
    for (int64_t t = (int64_t)blockIdx.x * kModelBlock + threadIdx.x; t < n && t < kModelStride; t += (int64_t)gridDim.x * kModelBlock) {
        double a = 0.0, b = 0.0;
        for (int64_t v = t; v < n; v += kModelStride) {
            unsigned long long sum_v = ell[v];
            if (slices.count) {
                const uint32_t bin = (uint32_t)(v >> slices.log2);
                if (slices.start[bin + 1u] - slices.start[bin] <= slices.part)
#pragma unroll
                    for (uint32_t i = 0; i < kModelSlices - 1u; ++i) sum_v += slices.more[(size_t)i * n + v];
            }
            const double l = (double)sum_v / kFix;
            const double q0 = (double)q[v];
            const double q1 = q0 - (1.0 - q0) * expm1(-l);
            q[v] = (float)q1;
            ell[v] = 0ull;
            a += q1;
            b += q1 * (1.0 - q1);
            if (COUNT && q1 > 0.0) sum[COUNT ? 2 : 0] += rows.work(v);
        }
        sum[0] += (unsigned long long)(a * kFix);
        sum[1] += (unsigned long long)(b * kFix);
    }
    add_sums<kModelBlock>(sums, sum);
}

// results of the size model left on the device: out[0..H] = mean, out[H+1..2H+1] = sigma (sums: per hop {sum q, sum q(1-q)} in 2^-32 units)
__global__ void k_model_finish(const unsigned long long *sums, int32_t num_hops, int32_t batch, double *out)
{
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    out[0] = (double)batch;
    out[num_hops + 1] = 0.0;
    for (int h = 0; h < num_hops; ++h) {
        out[h + 1] = (double)sums[2 * h] / kFix;
        out[num_hops + 1 + h + 1] = sqrt((double)sums[2 * h + 1] / kFix);
    }
}

// Scratch of zg_envelope_model_graph_static: the per-vertex log-sums (8 bytes) and probabilities (4 bytes) for up to
// ZG_STATIC_MODEL_MAX_NODES vertices plus the per-hop sums.  One copy per GPU, held until the process ends; host code
// never uses the array's name as an address, only what hipGetSymbolAddress returns for the current device.
constexpr size_t kStaticEllBytes = (size_t)ZG_STATIC_MODEL_MAX_NODES * 8;
constexpr size_t kStaticQBytes = (size_t)ZG_STATIC_MODEL_MAX_NODES * 4;
constexpr size_t kStaticSumsBytes = 2 * ZG_MAX_HOPS * 8;
static __device__ __align__(256) unsigned char scratch[kStaticEllBytes + kStaticQBytes + kStaticSumsBytes];

// How the sweep's edges are binned, laid out behind `used` bytes of the caller's buffer; bins == 0: they are not.  About 256 to 512
// bins, of up to 8192 vertices (64 KB of sums: two workgroups to a compute unit), beyond 16 M vertices of 16384; half as many where eight workgroups share
// a bin.  A thousand chunks, of at most 65536 edges (of 262144 with 1024 bins or more: their places are read a line each) unless their
// counters would be more than a byte per edge.  Below ZG_MODEL_BIN_EDGES edges never (see model_bins_work).
ModelBins model_bins(const zg_graph_t *g, void *temp, size_t used, size_t temp_bytes)
{
    ModelBins m;
    std::memset(&m, 0, sizeof(m));
    const int64_t n = g->num_nodes, E = g->num_edges;
    if (E < ZG_MODEL_BIN_EDGES || E >= ((int64_t)1 << 32)) return m;
    uint32_t log2;
    int64_t bins, chunk, part, parts;
    auto cut = [&](uint32_t slices) {
        log2 = 8;
        while (log2 < (slices > 1 ? 14 : 13) && (n >> log2) >= (slices > 1 ? 256 : 512)) ++log2;
        while (log2 < 14 && (n >> log2) >= 2048) ++log2;
        bins = (n + ((int64_t)1 << log2) - 1) >> log2;
        const int64_t want = std::max<int64_t>(4 * bins, std::min<int64_t>(bins >= 1024 ? 262144 : 65536, E / 1024));
        chunk = (want + kModelWindow - 1) / kModelWindow * kModelWindow;
        part = std::max<int64_t>(kModelMinPart, 2 * E / std::max<int64_t>(bins, 256));
        parts = bins + E / part;
    };
    auto lay_out = [&](bool terms, uint32_t slices) { // with the terms in the entries
        cut(slices);
        uint32_t block_log2 = terms ? 31 : 32 - log2;
        if (slices > 1)
            while (block_log2 > 0 && (n >> block_log2) < 8 * slices) --block_log2;
        const int64_t blocks = ((n - 1) >> block_log2) + 1, chunks = E / chunk + blocks;
        size_t at = used;
        auto place = [&](size_t bytes) {
            at = (at + kAlign - 1) / kAlign * kAlign;
            at += bytes;
            return static_cast<char *>(temp) + (at - bytes);
        };
        m.entry = place((size_t)E * (terms ? 8 : 4));
        m.term = terms ? nullptr : reinterpret_cast<unsigned long long *>(place((size_t)n * 8));
        m.slices = slices;
        m.more = reinterpret_cast<unsigned long long *>(place((size_t)(slices - 1) * n * 8));
        m.place = reinterpret_cast<uint32_t *>(place((size_t)(bins * chunks) * 4));
        m.start = reinterpret_cast<uint32_t *>(place((size_t)(bins + 1) * 4));
        m.share = reinterpret_cast<uint32_t *>(place((size_t)parts * 4));
        m.first_chunk = reinterpret_cast<uint32_t *>(place((size_t)(blocks + 1) * 4));
        m.chunk_edge = reinterpret_cast<uint32_t *>(place((size_t)(chunks + 1) * 4));
        m.sums = reinterpret_cast<unsigned long long *>(place((size_t)2 * ZG_MAX_HOPS * 8));
        m.block_log2 = block_log2;
        m.blocks = (uint32_t)blocks;
        m.chunks = (uint32_t)chunks;
        return at <= temp_bytes && (terms || bins <= kModelBinBlock); // (a thread of k_model_bin per bin)
    };
    const bool rows = n <= kModelRowsNodes ? lay_out(false, 1) : n <= kModelRowsNodes * kModelSlices && lay_out(false, kModelSlices);
    if (!rows && !lay_out(true, 1)) return m;
    if (bins > (int64_t)kModelMaxBins) return m;
    m.idx = g->d_indices;
    m.num_edges = E;
    m.num_nodes = n;
    m.log2 = log2;
    m.chunk = (uint32_t)chunk;
    m.part = (uint32_t)part;
    m.parts = (uint32_t)parts;
    m.bins = (uint32_t)bins;
    return m;
}

// Work of a sweep by atomics, in edges (46 ps each where they spread over the graph, up to 110 on a power law's hubs: 65 here; a row with a
// term is one more), that takes as long as the same sweep by bins, with `hops` sweeps to share the price of the places.  A sweep by bins takes
// 9 ps per edge, 12 us, and 4 us for every 512 vertices that a workgroup passes by; the places take 24 us.  Atomics / bins in us, uniform
// seeds.  Even graphs, one hop and three: 4 k vertices and 2^18 edges 44 / 62, 123 / 140; 30 k and 2^19 59 / 66, 167 / 153; 30 k and 2^20 84 / 76,
// 242 / 167; 1 M and 2^19 93 / 120, 268 / 305; 1 M and 2^20 108 / 105, 307 / 248; 8 M and 2^20 206 / 286, 577 / 769; 8 M and 2^21 284 / 231, 809 / 600.
// Power laws of skew 0.65: 40 k and 316 k edges 52 / 73, 148 / 149; 40 k and 473 k 66 / 73, 188 / 146; 10 k and 482 k 73 / 75, 209 / 152; 80 k and 0.6 M
// 78 / 74, 224 / 160.  2.4 M vertices and 115 M edges, one hop: 1.1 ms by bins; by atomics 0.11, 0.55, 0.94, 1.3 ms with 1, 10, 18, 25 % of the
// vertices as seeds, 5.6 with all; three hops from 1 % 2.2 ms, 3.0 all by bins.  (All with 8-byte entries.  With terms by row the places take
// 6 ps per edge more and a sweep 4 to 6 less: 90 k vertices and 1 M edges, one hop, 81 to 85 us with either.)
// The line is that of 8-byte entries, and of seeds that are drawn evenly.  With terms by row, where further hops go by bins anyway, it lies too high: 2.4 M vertices
// and 111 M edges, seeds from 3 to 13 % of the vertices, us now / all by bins: one hop 1146 to 1576 / 940, two 2265 to 2696 / 1270, three 2601 to 3033 /
// 1600; from 16 % on, and for 1 % in one hop, the better of the two.  40 k and 2.2 M, 10 to 25 %, two hops 172 to 215 / 134; 8 M and 119 M (8-byte entries), 5 to 13 %, one
// hop 1948 to 3262 / 1620, two 3743 to 4835 / 2950.
int64_t model_bins_work(const ModelBins &m, int hops)
{
    return m.num_edges / 7 + 180000 + 360000 / hops + 120 * m.num_nodes / m.chunks;
}

template <typename OffT>
void enqueue_model_bin(const zg_graph_t *g, const ModelBins &m, const float *q, int32_t fanout, int32_t replace, hipStream_t st)
{
    const OffT *off = static_cast<const OffT *>(g->d_offsets);
    const size_t lds = (size_t)m.bins * 4;
    if (m.term)
        hipLaunchKernelGGL((k_model_bin<OffT, false>), dim3(m.chunks), dim3(kModelBinBlock), lds, st, m, off, q, fanout, replace);
    else
        hipLaunchKernelGGL((k_model_bin<OffT, true>), dim3(m.chunks), dim3(kModelBinBlock), lds, st, m, off, q, fanout, replace);
}

// once per call: places for the edges, and the edges themselves unless their entries hold a hop's terms
template <typename OffT>
void enqueue_model_places(const zg_graph_t *g, const ModelBins &m, hipStream_t st)
{
    hipLaunchKernelGGL(k_model_chunks<OffT>, dim3(1), dim3(1024), (size_t)m.blocks * 4, st, m, static_cast<const OffT *>(g->d_offsets));
    hipLaunchKernelGGL(k_model_count, dim3(m.chunks), dim3(1024), (size_t)m.bins * 4, st, m);
    hipLaunchKernelGGL(k_model_places, dim3(m.bins), dim3(256), 0, st, m);
    hipLaunchKernelGGL(k_model_starts, dim3(1), dim3(1024), 0, st, m);
    if (m.term) enqueue_model_bin<OffT>(g, m, nullptr, 0, 0, st);
}

// one hop by bins: the terms, their sums
template <typename OffT>
void enqueue_model_sums(const zg_graph_t *g, const ModelBins &m, const float *q, unsigned long long *ell, int32_t fanout, int32_t replace, hipStream_t st)
{
    const int64_t n = g->num_nodes;
    const size_t lds = (size_t)8 << m.log2;
    if (m.term) {
        hipLaunchKernelGGL(k_model_terms<OffT>, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, static_cast<const OffT *>(g->d_offsets), q, m.term,
                           n, fanout, replace);
        hipLaunchKernelGGL(k_model_add<false>, dim3(m.parts * m.slices), dim3(kModelAddBlock(false)), lds, st, m, ell);
    } else {
        enqueue_model_bin<OffT>(g, m, q, fanout, replace, st);
        hipLaunchKernelGGL(k_model_add<true>, dim3(m.parts), dim3(kModelAddBlock(true)), lds, st, m, ell);
    }
}

// the sweep over the vertices that starts the size model
void enqueue_model_init(const zg_graph_t *g, float *q, unsigned long long *ell, const float *seed_prob, int32_t batch, const ModelRows &rows, unsigned long long *work,
                        hipStream_t st)
{
    const int64_t n = g->num_nodes;
    const float uniform = (float)((double)batch / (double)n);
    if (rows.off)
        hipLaunchKernelGGL(k_model_init<true>, dim3((unsigned)std::min<int64_t>(kModelGrid, (n + kModelBlock - 1) / kModelBlock)), dim3(kModelBlock), 0, st, q, ell,
                           seed_prob, uniform, n, rows, work);
    else
        hipLaunchKernelGGL(k_model_init<false>, dim3((unsigned)std::min<int64_t>(1 << 16, (n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, q, ell, seed_prob, uniform,
                           n, rows, work);
}

// one hop of it: the sweep over the edges and the update of the probabilities
struct ModelHop {
    float *q;
    unsigned long long *ell, *sums;
    int32_t fanout, replace;
    bool binned;
    ModelGate gate;
    ModelRows rows; // `off` not null: sums[2] is the work of the next hop
};

void enqueue_model_hop(const zg_graph_t *g, const ModelBins &m, const ModelHop &a, hipStream_t st)
{
    const int64_t n = g->num_nodes;
    const bool wide = g->offsets_dtype == ZG_I64;
    if (a.binned) {
        if (wide)
            enqueue_model_sums<int64_t>(g, m, a.q, a.ell, a.fanout, a.replace, st);
        else
            enqueue_model_sums<int32_t>(g, m, a.q, a.ell, a.fanout, a.replace, st);
    } else {
        int32_t rows = 1;
        while (rows < 64 && n / (2 * rows) >= kModelPushWaves) rows *= 2;
        const int64_t waves = (n + rows - 1) / rows;
        const dim3 grid((unsigned)std::min<int64_t>(1 << 16, (waves + (kBlock / 64) - 1) / (kBlock / 64)));
        if (wide)
            hipLaunchKernelGGL(k_model_push<int64_t>, grid, dim3(kBlock), 0, st, (const int64_t *)g->d_offsets, g->d_indices, a.q, a.ell, n, a.fanout, a.replace,
                               rows, a.gate);
        else
            hipLaunchKernelGGL(k_model_push<int32_t>, grid, dim3(kBlock), 0, st, (const int32_t *)g->d_offsets, g->d_indices, a.q, a.ell, n, a.fanout, a.replace,
                               rows, a.gate);
    }
    const dim3 sweep((unsigned)std::min<int64_t>(kModelGrid, (n + kModelBlock - 1) / kModelBlock));
    const ModelSlices slices = {m.more, a.binned && m.slices > 1 ? m.slices - 1u : 0u, m.start, m.log2, m.part};
    if (a.rows.off)
        hipLaunchKernelGGL(k_model_update<true>, sweep, dim3(kModelBlock), 0, st, a.q, a.ell, n, a.sums, a.gate, a.rows, slices);
    else
        hipLaunchKernelGGL(k_model_update<false>, sweep, dim3(kModelBlock), 0, st, a.q, a.ell, n, a.sums, a.gate, a.rows, slices);
}

#define ZG_HIP(call)                                                                                         \
    do {                                                                                                     \
        hipError_t e_ = (call);                                                                              \
        if (e_ != hipSuccess) return fail(ZG_EHIP, std::string(#call) + ": " + hipGetErrorString(e_));       \
    } while (0)

int validate_graph_device(const zg_graph_t *g)
{
    uint32_t *d_bad = nullptr;
    ZG_HIP(hipMalloc(&d_bad, 4));
    hipError_t e = hipMemset(d_bad, 0, 4);
    if (e == hipSuccess) {
        const int grid = (int)std::min<int64_t>(65535, (g->num_nodes + 255) / 256);
        if (g->offsets_dtype == ZG_I64)
            k_validate<int64_t><<<grid, 256>>>((const int64_t *)g->d_offsets, g->d_indices, g->num_nodes, d_bad);
        else
            k_validate<int32_t><<<grid, 256>>>((const int32_t *)g->d_offsets, g->d_indices, g->num_nodes, d_bad);
        e = hipGetLastError();
    }
    uint32_t bad = 0;
    if (e == hipSuccess) e = hipMemcpy(&bad, d_bad, 4, hipMemcpyDeviceToHost);
    (void)hipFree(d_bad);
    if (e != hipSuccess) return fail(ZG_EHIP, std::string("graph validation: ") + hipGetErrorString(e));
    if (bad & 1u) return fail(ZG_EINVAL, "graph validation: a neighbor id is out of range");
    if (bad & 2u) return fail(ZG_EINVAL, "graph validation: a row is not strictly ascending");
    return ZG_OK;
}

} // namespace zg

// =================================================================================================
// plan
// =================================================================================================
using namespace zg;

struct zg_plan_s {
    const zg_graph_t *graph = nullptr;
    Layout lay;
    char *ws = nullptr;
    uint32_t flags = 0;
    int32_t batch = 0;
    int device = -1;
    const float *d_feat = nullptr;
    int64_t ld_feat = 0;
    Mailbox *mailbox = nullptr;     // pinned host memory
    Mailbox *mailbox_dev = nullptr; // the same memory as the device addresses it
    uint32_t issued = 0;            // steps enqueued so far (mod 2^32, like the device-side step counter)
    hipStream_t last_stream = nullptr; // stream of the last enqueued step (what zg_plan_destroy waits for)
    bool stepped = false;
    bool recorded = false;          // a step is part of a caller's graph
    bool broken = false;            // a step was enqueued in part
    zg_plan_s *twin = nullptr;      // worst-case twin (ZG_PLAN_SAFE_TWIN): own outputs, metadata and mailbox, shared scratch
    hipStream_t own_stream = nullptr;
    hipGraph_t graph_obj = nullptr; // (plans that replay one: see issue_step)
    hipGraphExec_t graph_exec = nullptr;

    Drmb *drmb() const { return reinterpret_cast<Drmb *>(ws + lay.off_drmb); }
    uint32_t *log() const { return reinterpret_cast<uint32_t *>(ws + lay.off_log); }
    int32_t *S() const { return reinterpret_cast<int32_t *>(ws + lay.off_S); }
    int32_t *row_ptr(int h) const { return reinterpret_cast<int32_t *>(ws + lay.off_row_ptr[h]); }
    int32_t *nbr(int h) const { return reinterpret_cast<int32_t *>(ws + lay.off_nbr[h]); }
    int32_t *col(int h) const { return reinterpret_cast<int32_t *>(ws + lay.off_col[h]); }
    float *X() const { return lay.feat_dim > 0 ? reinterpret_cast<float *>(ws + lay.off_X) : nullptr; }
    float *agg() const { return lay.feat_dim > 0 ? reinterpret_cast<float *>(ws + lay.off_agg) : nullptr; }
    int32_t *local_id() const { return reinterpret_cast<int32_t *>(ws + lay.off_local_id); }
    uint32_t *bitmap(int hop) const { return reinterpret_cast<uint32_t *>(ws + lay.off_bitmap[hop & 1]); } // the one hop `hop` fills
    uint32_t *seen() const { return reinterpret_cast<uint32_t *>(ws + lay.off_seen); }
    uint64_t *status() const { return reinterpret_cast<uint64_t *>(ws + lay.off_status); }
    uint8_t *own() const { return reinterpret_cast<uint8_t *>(ws + lay.off_own); }
    uint64_t *status_cnt(int l) const { return reinterpret_cast<uint64_t *>(ws + lay.off_status_cnt[l]); }
    uint64_t *status_edge(int l) const { return reinterpret_cast<uint64_t *>(ws + lay.off_status_edge[l]); }
};

namespace {

RelabelArgs relabel_args(const zg_plan_t *p, int hop, bool present, const zg_plan_t *gate = nullptr)
{
    RelabelArgs ra;
    std::memset(&ra, 0, sizeof(ra));
    ra.gate = gate ? gate->drmb() : nullptr;
    if (!present) return ra;
    ra.drmb = p->drmb();
    ra.nbr = p->nbr(hop);
    ra.local_id = p->local_id();
    ra.col = p->col(hop);
    ra.num_nodes = (uint32_t)p->graph->num_nodes;
    ra.hop = hop;
    ra.blocks = (uint32_t)((p->lay.edge_cap[hop] + kRelabelPerBlock - 1) / kRelabelPerBlock);
    return ra;
}

// Whether the step's aggregation reads the feature table and writes the newly discovered vertices' rows of X on the way
// ("one pass"), instead of the gather copying every row of S_{H-1} and the aggregation reading X ("two passes").
// ZG_PLAN_FUSED_INPUT does not materialise those rows at all.  One pass moves up to a third less memory traffic and has
// one launch fewer.  Measured on MI355X against two passes (step time on one stream / with four plans in flight):
// 56 GB table of 512-byte rows -6 % with four plans; 0.6 GB table of 2400-byte rows -7 % / -3 %; 1 GB of 400-byte rows
// -4 % / 0; 1 GB of 1 KB rows 0 / -1 %.  Hence one pass unless the flag asks for two.
bool x_written_by_aggregation(const zg_plan_t *p)
{
    if (!p->d_feat || p->lay.feat_dim <= 0 || (p->flags & ZG_PLAN_FUSED_INPUT)) return false;
    return (p->flags & ZG_PLAN_X_TWO_PASS) == 0;
}

// One pass (and ZG_PLAN_FUSED_INPUT): how the rows move.  The table's rows are loaded through the caches - about a fifth of
// the last hop's edges lead to a vertex another edge leads to as well, and its row is then found in the last-level cache
// instead of in HBM.  What the feature launches write - the frontier's rows of X, the new vertices' rows of X, the rows of
// means - nothing in the step reads again: it is stored non-temporally, whatever the row length (rows that are not whole
// 128-byte lines gain as much: 2400-byte rows 84 -> 71 us per step with four plans in flight, 400-byte rows 64 -> 59 us).
// Measured at a 56 GB table of 512-byte rows, step time with four plans in flight / on one stream: table loads and all stores
// non-temporal 183 / 215 us (X rows of new vertices only: 191 / 222 us), loads cached and stores non-temporal 174 / 214 us,
// both cached 194 / 242 us.

// (`blocks_before` of the last launch do something else)
FinishArgs finish_args(const zg_plan_t *p, bool present, const zg_plan_t *gate = nullptr, bool defer_completed = false, bool enqueued = false,
                       uint32_t blocks_before = 0)
{
    FinishArgs fa;
    std::memset(&fa, 0, sizeof(fa));
    if (!present) return fa;
    const int H = p->lay.num_hops;
    fa.drmb = p->drmb();
    fa.gate = gate ? gate->drmb() : nullptr;
    fa.gate_mailbox = gate ? gate->mailbox_dev : nullptr;
    fa.defer_completed = defer_completed ? 1 : 0;
    fa.enqueued = enqueued ? 1 : 0;
    fa.mailbox = p->mailbox_dev;
    fa.S = p->S();
    fa.seen = p->seen();
    fa.log = p->log();
    fa.status = p->status();
    fa.status_words = p->lay.status_words;
    fa.num_hops = H;
    fa.blocks = (uint32_t)((p->lay.node_cap[H - 1] + kBlock - 1) / kBlock);
    // A read of host memory: in the first workgroup, where others are still to come when it has ended; in a launch that the chip holds at once, in
    // the last one, which has little else to do.
    fa.prefetch = blocks_before < 1024u ? blocks_before + fa.blocks - 1u : 0u;
    return fa;
}

RowArgs gather_args(const zg_plan_t *p, const float *d_feat, int64_t ld, int32_t dim, float *d_out, int64_t ld_out, int hop_rows)
{
    RowArgs a;
    std::memset(&a, 0, sizeof(a));
    const RowTiling t = gather_tiling(dim);
    a.src = d_feat;
    a.dst = d_out;
    a.S = p->S();
    a.n_rows = &p->drmb()->n[hop_rows];
    a.ld_src = ld;
    a.ld_dst = ld_out;
    a.inv = t.inv;
    a.dimv = t.dimv;
    a.last = (uint32_t)(dim - t.vec);
    a.vec4 = t.vec == 4 ? 1 : 0;
    a.rows = t.rows;
    a.blocks = (uint32_t)((p->lay.node_cap[hop_rows] + t.rows - 1) / t.rows);
    return a;
}

// input rows addressed by `col` (local ids, bounded by n[hop+1]) or, with by_gid, by nbr_gid (global ids into the table)
RowArgs aggregate_args(const zg_plan_t *p, int hop, const float *d_in, int64_t ld_in, int32_t dim, float *d_out, int64_t ld_out,
                       bool by_gid)
{
    RowArgs a;
    std::memset(&a, 0, sizeof(a));
    const RowTiling t = aggregate_tiling(dim);
    a.src = d_in;
    a.dst = d_out;
    a.row_ptr = p->row_ptr(hop);
    a.col = by_gid ? p->nbr(hop) : p->col(hop);
    a.n_rows = &p->drmb()->n[hop];
    a.n_cols = &p->drmb()->n[hop + 1];
    a.col_limit = (uint32_t)p->graph->num_nodes;
    a.ld_src = ld_in;
    a.ld_dst = ld_out;
    a.inv = t.inv;
    a.dimv = t.dimv;
    a.last = (uint32_t)(dim - t.vec);
    a.vec4 = t.vec == 4 ? 1 : 0;
    a.rows = t.rows;
    a.max_fanout = (uint32_t)p->lay.fanout[hop];
    a.blocks = (uint32_t)((p->lay.node_cap[hop] + t.rows - 1) / t.rows);
    return a;
}

// zg_step_timed: events to record right before and right after the aggregation launch of the plan's own step
struct StepProbe {
    hipEvent_t before, after;
    hipError_t error; // what recording them returned (the step is enqueued either way)
};

// Where a step's launches go, and how many of them have gone there.  (What a launch returned, and not hipGetLastError: that may be an earlier
// error of the caller's own.  An error that was returned does not stay behind for the caller's next launch.)
struct Queue {
    hipStream_t st;
    bool recorded = false; // into a caller's graph
    int launched = 0;
    template <class... P> int launch(void (*kernel)(P...), unsigned grid, unsigned block, size_t lds, P... a)
    {
        void *args[] = {&a...};
        const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block), args, lds, st);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(ZG_EHIP, std::string("hipLaunchKernel: ") + hipGetErrorString(e));
        }
        ++launched;
        return ZG_OK;
    }
};

int launch_gather(const RowArgs &gat, const RelabelArgs &ra, Queue &q)
{
    const unsigned grid = gat.blocks + ra.blocks;
    if (grid == 0) return ZG_OK;
    return q.launch(gat.vec4 ? k_gather<4> : k_gather<1>, grid, kBlock, (size_t)kBlock * 4, gat, ra);
}

int launch_aggregate(const RowArgs &agg, const FinishArgs &fa, Queue &q, const RowArgs *copy = nullptr)
{
    const unsigned grid = agg.blocks + fa.blocks + (copy ? copy->blocks : 0u);
    if (grid == 0) return ZG_OK;
    size_t lds = agg.blocks ? ((size_t)agg.rows + 1 + (size_t)agg.rows * agg.max_fanout * (agg.x_dst ? 2 : 1)) * 4 : 0;
    if (copy) lds = std::max(lds, (size_t)copy->rows * 4);
    if (copy) return q.launch(agg.vec4 ? k_aggregate<4, RowArgs> : k_aggregate<1, RowArgs>, grid, kBlock, lds, agg, fa, *copy);
    return q.launch(agg.vec4 ? k_aggregate<4, NoCopy> : k_aggregate<1, NoCopy>, grid, kBlock, lds, agg, fa, NoCopy());
}

// How the last hop's new vertices carry their marking edge's tag, where that hop marks bytes (all zero: they do not).  A plan and
// its twin share one id map, and the replayed aggregation of one may meet the other's entries: both read them by one layout, whether
// their own hop marks bytes (tags) or bits (tag 0).
MarkTag mark_tag(const zg_plan_t *p)
{
    const Layout &L = p->lay;
    MarkTag t = {0, 0u, 0u};
    if (!x_written_by_aggregation(p)) return t;
    int lid_bits = 1;
    while (lid_bits < 31 && ((int64_t)1 << lid_bits) < L.id_rows) ++lid_bits;
    const int bits = std::min(7, 31 - lid_bits);
    if (bits <= 0) return t; // no room for a tag: every edge to a new vertex writes its row
    t.shift = 31 - bits;
    t.mask = (1u << bits) - 1u;
    const int64_t row = (int64_t)L.feat_dim * 4;
    t.reach_rows = (uint32_t)((reach_bytes(row) + row - 1) / row);
    return t;
}

// The step's two feature launches.  Two passes: the gather copies every row of S_{H-1} into X and the mean reads X.
// One pass (and ZG_PLAN_FUSED_INPUT): the gather copies the rows of the frontier D_{H-1} only; the mean reads its input
// rows from the table, addressed by the sampled global ids (feat[nbr_gid[e]] is the row X[col[e]] holds), and - unless
// ZG_PLAN_FUSED_INPUT leaves them out - writes the other rows of X, those of the last hop's newly discovered
// vertices, on the way.
void step_feature_args(const zg_plan_t *p, RowArgs *gat, RowArgs *agg)
{
    const Layout &L = p->lay;
    const int H = L.num_hops;
    const bool fused = (p->flags & ZG_PLAN_FUSED_INPUT) != 0, one_pass = x_written_by_aggregation(p);
    if (fused || one_pass) {
        *agg = aggregate_args(p, H - 1, p->d_feat, p->ld_feat, L.feat_dim, p->agg(), L.ld_out, true);
        // the aggregation relabels the last hop's edges itself (it holds their sampled ids anyway): no launch in between
        agg->local_id = p->local_id();
        agg->col_out = p->col(H - 1);
    } else {
        *agg = aggregate_args(p, H - 1, p->X(), L.ld_out, L.feat_dim, p->agg(), L.ld_out, false);
    }
    if (one_pass) {
        agg->x_dst = p->X();
        agg->ld_x = L.ld_out;
        agg->own = L.byte_marks[H - 1] ? nullptr : p->own();
        agg->tag = mark_tag(p);
    }
    if (fused || one_pass) agg->nt = 1;
    *gat = gather_args(p, p->d_feat, p->ld_feat, L.feat_dim, p->X(), L.ld_out, (fused || one_pass) ? H - 1 : H);
}

// whether the step has no gather launch of its own: the frontier's rows are copied by workgroups of the closing hop-kernel
// launch and the aggregation relabels the last hop's edges itself (H+2 launches per step)
bool features_ride_along(const zg_plan_t *p)
{
    return p->d_feat && p->lay.feat_dim > 0 && ((p->flags & ZG_PLAN_FUSED_INPUT) || x_written_by_aggregation(p));
}

template <typename OffT>
int launch_hop(const HopArgs &ha, const HopRoles &o, unsigned grid, size_t lds, Queue &q)
{
    const bool prev = ha.bytes_prev != 0, next = ha.bytes_next != 0;
    if (ha.launch == 0) return q.launch(next ? k_hop<OffT, true, false, true> : k_hop<OffT, true, false, false>, grid, kHopBlock, lds, ha, o);
    if (prev) return q.launch(next ? k_hop<OffT, false, true, true> : k_hop<OffT, false, true, false>, grid, kHopBlock, lds, ha, o);
    return q.launch(next ? k_hop<OffT, false, false, true> : k_hop<OffT, false, false, false>, grid, kHopBlock, lds, ha, o);
}

// the sampling of a small step
int launch_small(const zg_plan_t *p, Queue &q, const StepInputs &in, const zg_plan_t *gate)
{
    const Layout &L = p->lay;
    const zg_graph_t *g = p->graph;
    SmallArgs sa;
    std::memset(&sa, 0, sizeof(sa));
    HopArgs &ha = sa.hop;
    ha.offsets = g->d_offsets;
    ha.indices = g->d_indices;
    ha.drmb = p->drmb();
    ha.gate = gate ? gate->drmb() : nullptr;
    ha.in = in;
    ha.mailbox = gate ? gate->mailbox_dev : p->mailbox_dev;
    ha.S = p->S();
    ha.local_id = p->local_id();
    ha.own = x_written_by_aggregation(p) ? p->own() : nullptr;
    ha.num_nodes = (uint32_t)g->num_nodes;
    ha.num_hops = L.num_hops;
    ha.replace = (p->flags & ZG_PLAN_REPLACE) ? 1 : 0;
    ha.batch = (uint32_t)p->batch;
    ha.stage_edges = (uint32_t)kSmallStage;
    for (int h = 0; h < L.num_hops; ++h) {
        sa.row_ptr[h] = p->row_ptr(h);
        sa.nbr[h] = p->nbr(h);
        sa.col[h] = p->col(h);
        sa.fanout[h] = (uint32_t)L.fanout[h];
        sa.edge_cap[h] = (uint32_t)L.edge_cap[h];
    }
    for (int h = 0; h <= L.num_hops; ++h) sa.cap[h] = (uint32_t)L.node_cap[h];
    sa.words = (uint32_t)(((g->num_nodes + 31) / 32 + 31) / 32 * 32);
    const size_t lds = (kSmallStage + 2 * (size_t)sa.words) * 4;
    return q.launch(g->offsets_dtype == ZG_I64 ? k_small<int64_t> : k_small<int32_t>, 1u, kHopBlock, lds, sa);
}

// LDS of a ranking workgroup of the closing launch: the vertices expanded, the tile's words, and these with their ranks; of a tile of more
// than a word per lane no ranks, and the words only out of mark bytes
size_t close_lds(const HopArgs &a)
{
    const size_t words = a.words_per_tile;
    return (size_t)kCloseBatch * 4 + (words <= (size_t)kCloseBlock ? words * 12 : a.bytes_prev ? words * 4 : 0);
}

// a whole step, in order, on one stream (a step's launches, or - captured once - those of a graph): the hop kernel's launches 0..H, then the
// two feature launches.  With `gate` the kernels are those of gate's worst-case twin `p`, run on gate's inputs and
// only if gate's step overflowed; `defer_completed` marks a plan whose gated twin follows in the same sequence.
int enqueue_body(const zg_plan_t *p, Queue &q, const StepInputs &in, const zg_plan_t *gate = nullptr, bool defer_completed = false,
                 StepProbe *probe = nullptr)
{
    const Layout &L = p->lay;
    const zg_graph_t *g = p->graph;
    const int H = L.num_hops;
    const bool feats = p->d_feat && L.feat_dim > 0;
    const bool enqueued = !gate && !q.recorded;
    const bool ride = features_ride_along(p);
    RowArgs agg, gat, no_rows;
    std::memset(&agg, 0, sizeof(agg));
    std::memset(&gat, 0, sizeof(gat));
    std::memset(&no_rows, 0, sizeof(no_rows));
    if (feats) step_feature_args(p, &gat, &agg);
    if (L.small) {
        const int rc = launch_small(p, q, in, gate);
        if (rc != ZG_OK) return rc;
    }
    for (int l = 0; l <= H && !L.small; ++l) {
        HopArgs ha;
        std::memset(&ha, 0, sizeof(ha));
        ha.offsets = g->d_offsets;
        ha.indices = g->d_indices;
        ha.drmb = p->drmb();
        ha.gate = gate ? gate->drmb() : nullptr;
        ha.in = in;
        ha.mailbox = gate ? gate->mailbox_dev : p->mailbox_dev;
        ha.S = p->S();
        ha.local_id = p->local_id();
        ha.marks_prev = l > 0 ? p->bitmap(l - 1) : nullptr;
        ha.marks_next = l < H ? p->bitmap(l) : nullptr;
        ha.seen = p->seen();
        ha.row_ptr = l < H ? p->row_ptr(l) : nullptr;
        ha.nbr = l < H ? p->nbr(l) : nullptr;
        ha.bytes_prev = l > 0 ? L.byte_marks[l - 1] : 0;
        ha.bytes_next = l < H ? L.byte_marks[l] : 0;
        if (l == H - 1 && x_written_by_aggregation(p)) {
            ha.own = ha.bytes_next ? nullptr : p->own();
            ha.tag_next = ha.bytes_next;
        }
        if (l == H) ha.tag = mark_tag(p);
        ha.status_cnt = p->status_cnt(l);
        ha.status_edge = p->status_edge(l);
        ha.max_tickets = (uint32_t)L.max_tickets;
        ha.num_nodes = (uint32_t)g->num_nodes;
        ha.launch = l;
        ha.num_hops = H;
        ha.fanout = l < H ? L.fanout[l] : 1;
        ha.rows_per_wave = 64u / (uint32_t)ha.fanout;
        ha.inv_fanout = 65536u / (uint32_t)ha.fanout + 1u;
        ha.replace = (p->flags & ZG_PLAN_REPLACE) ? 1 : 0;
        ha.rows_per_ticket = l < H ? (uint32_t)(sample_tile_nodes(L.fanout[l]) * L.old_tpt[l]) : 256u;
        ha.cap_rows = (uint32_t)L.node_cap[l];
        ha.edge_cap = l < H ? (uint32_t)L.edge_cap[l] : 0u;
        ha.words_per_tile = l > 0 ? (uint32_t)L.tile_words[l] : (uint32_t)kHopMinTileWords;
        ha.chunk_log2 = 5; // as few vertices per lane as the workgroup has lanes for
        while (ha.chunk_log2 > 2 && ((uint64_t)ha.words_per_tile << (6 - ha.chunk_log2)) <= (uint64_t)(l < H ? kHopBlock : kCloseBlock)) --ha.chunk_log2;
        ha.rank_tiles = (uint32_t)L.rank_tiles[l];
        ha.batch = (uint32_t)p->batch;
        // Tickets: see k_hop.  A tile ranked by pieces changes its marks before its totals are out: nobody else can work them out.
        const bool by_pieces = l > 0 && L.tile_words[l] > (l < H ? kHopBlock : kCloseBlock);
        ha.draw = by_pieces;
        ha.patience = by_pieces ? kSpinLimit : (p->flags & ZG_PLAN_IMPATIENT) ? 0u : kPatience;
        ha.blocks = (uint32_t)(L.old_tickets[l] + L.rank_tiles[l]);
        int rc;
        // the edges of hop l-2 can be relabeled now: launch l-1 ranked the last vertices they point to
        const RelabelArgs ra = relabel_args(p, l - 2, l >= 2);
        IngestArgs ia;
        std::memset(&ia, 0, sizeof(ia));
        if (l == 0) {
            ia.in = in;
            ia.drmb = p->drmb();
            ia.gate = ha.gate;
            ia.mailbox = ha.mailbox;
            ia.S = p->S();
            ia.local_id = p->local_id();
            ia.seen = p->seen();
            ia.batch = (uint32_t)p->batch;
            ia.num_nodes = (uint32_t)g->num_nodes;
            ia.blocks = (uint32_t)((p->batch + kHopBlock - 1) / kHopBlock);
        }
        if (l == H) {
            // the closing launch can carry the copy of the frontier's rows: D_{H-1} is final since launch H-1
            // (as many rows to a workgroup as its lanes load at once: with twice as many 60 k rows of 400 bytes 20.3 us instead of 19.0, 300-byte rows
            // 17.8 instead of 16.0)
            CloseRoles roles = {ra, ride ? gat : no_rows};
            if (ha.bytes_prev) roles.rel.tag = ha.tag;
            roles.gat.blocks = ride ? (uint32_t)((L.node_cap[H - 1] + roles.gat.rows - 1) / roles.gat.rows) : 0u;
            const size_t lds = std::max(close_lds(ha), ride ? ((size_t)roles.gat.rows * 2 + 1) * 4 : 0);
            rc = q.launch(ha.bytes_prev ? k_close<true> : k_close<false>, ha.blocks + ra.blocks + roles.gat.blocks, kCloseBlock, lds, ha, roles);
        } else {
            const HopRoles roles = {ra, ia};
            const unsigned grid = ha.blocks + ra.blocks + ia.blocks;
            // The dynamic LDS: ids on their way, a bit-marking pass's dedup set, a ranking tile's words.  As many ids as leave room
            // for two workgroups on a compute unit (a tile of 16 words per lane: one), at least 4096 - 64 rows of any fanout.
            const size_t words = (l > 0 ? ha.words_per_tile : 0u) + (!ha.bytes_next ? (uint32_t)kSampleHashSlots : 0u);
            const size_t room = kHopLdsBytes / 4 - sizeof(HopShared) / 4;
            ha.stage_edges = (uint32_t)std::min<size_t>(kHopMaxStage, room > words + kHopMinStage ? (room - words) / 64 * 64 : kHopMinStage);
            const size_t lds = (ha.stage_edges + words) * 4u;
            rc = g->offsets_dtype == ZG_I64 ? launch_hop<int64_t>(ha, roles, grid, lds, q) : launch_hop<int32_t>(ha, roles, grid, lds, q);
        }
        if (rc != ZG_OK) return rc;
    }
    // the tail: {gather + relabel of the last hop} - unless both ride along elsewhere -, then {aggregation + end-of-step
    // clean-up}.  (One launch for all four roles was measured: no gain - the two big roles are bound by the same memory fabric.)
    if (!feats) {
        const RelabelArgs ra = relabel_args(p, H - 1, true, gate);
        const FinishArgs fa = finish_args(p, true, gate, defer_completed, enqueued, ra.blocks);
        return q.launch(k_tail, ra.blocks + fa.blocks, kBlock, 0, ra, fa);
    }
    if (!ride) {
        int rc = launch_gather(gat, relabel_args(p, H - 1, true, gate), q);
        if (rc != ZG_OK) return rc;
    }
    // a small step's frontier rows are copied by workgroups of the aggregation launch - by a launch of their own, ahead of it, where
    // the events are to bracket the aggregation alone
    const bool copy_along = L.small && ride && !probe;
    if (L.small && ride && probe) {
        const int rc = launch_gather(gat, relabel_args(p, 0, false), q);
        if (rc != ZG_OK) return rc;
    }
    if (probe) probe->error = hipEventRecord(probe->before, q.st);
    const FinishArgs fa = finish_args(p, true, gate, defer_completed, enqueued, agg.blocks + (copy_along ? gat.blocks : 0u));
    int rc = launch_aggregate(agg, fa, q, copy_along ? &gat : nullptr);
    if (rc == ZG_OK && probe && probe->error == hipSuccess) probe->error = hipEventRecord(probe->after, q.st);
    return rc;
}

// the plan's step, followed - with ZG_PLAN_AUTO_FALLBACK - by its twin's step behind the device-side gate
int enqueue_step(const zg_plan_t *p, Queue &q, const StepInputs &in, StepProbe *probe = nullptr)
{
    const bool autofb = (p->flags & ZG_PLAN_AUTO_FALLBACK) && p->twin;
    int rc = enqueue_body(p, q, in, nullptr, autofb, probe);
    if (rc == ZG_OK && autofb) rc = enqueue_body(p->twin, q, in, p, false);
    return rc;
}

void drop_graph(zg_plan_t *p)
{
    if (p->graph_exec) (void)hipGraphExecDestroy(p->graph_exec);
    if (p->graph_obj) (void)hipGraphDestroy(p->graph_obj);
    p->graph_exec = nullptr;
    p->graph_obj = nullptr;
}

bool replays_graph(const zg_plan_t *p) { return (p->flags & ZG_PLAN_AUTO_FALLBACK) && !(p->flags & ZG_PLAN_EAGER); }

int build_graph(zg_plan_t *p)
{
    drop_graph(p);
    if (!replays_graph(p) || !p->twin) return ZG_OK;
    ZG_HIP(hipStreamBeginCapture(p->own_stream, hipStreamCaptureModeThreadLocal));
    Queue q{p->own_stream};
    int rc = enqueue_step(p, q, StepInputs{nullptr, 0ull});
    hipGraph_t gobj = nullptr;
    hipError_t e = hipStreamEndCapture(p->own_stream, &gobj);
    if (rc != ZG_OK) {
        if (gobj) (void)hipGraphDestroy(gobj);
        return rc;
    }
    if (e != hipSuccess) return fail(ZG_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
    p->graph_obj = gobj;
    ZG_HIP(hipGraphInstantiate(&p->graph_exec, p->graph_obj, nullptr, nullptr, 0));
    return ZG_OK;
}

} // namespace

extern "C" {

static int make_plan_object(zg_plan_t **out, const zg_graph_t *g, const Layout &L, uint32_t flags, int32_t batch,
                            char *ws, hipStream_t st, bool init_scratch)
{
    zg_plan_t *p = new (std::nothrow) zg_plan_t();
    if (!p) return fail(ZG_ENOMEM, "out of host memory");
    p->graph = g;
    p->lay = L;
    p->ws = ws;
    p->flags = flags;
    p->batch = batch;
    auto bail = [&](int code) {
        zg_plan_destroy(p);
        return code;
    };
    if (hipGetDevice(&p->device) != hipSuccess) return bail(fail(ZG_EHIP, "hipGetDevice failed"));
    if (p->device != g->device) return bail(fail(ZG_ESTATE, "current device differs from the graph's device"));
    {
        void *host = nullptr, *dev = nullptr;
        if (hipHostMalloc(&host, sizeof(Mailbox), hipHostMallocDefault) != hipSuccess)
            return bail(fail(ZG_ENOMEM, "hipHostMalloc of the step mailbox failed"));
        std::memset(host, 0, sizeof(Mailbox));
        p->mailbox = static_cast<Mailbox *>(host);
        if (hipHostGetDevicePointer(&dev, host, 0) != hipSuccess) return bail(fail(ZG_EHIP, "hipHostGetDevicePointer failed"));
        p->mailbox_dev = static_cast<Mailbox *>(dev);
    }
    // A stream of the plan's own, for the capture of a graph - and where there is none all the same: the runtime spreads a process's streams over
    // four hardware queues as they are made, and callers with a stream per plan and the default one have five.  Which of them share a queue
    // is the runtime's affair and depends on what else the process makes; with these in between it came out better.  (110 M vertices, four plans on
    // four streams, a step of each, without / with: streams made before the plans 943 / 857 us, behind them 980 / 906.)  A plan made with
    // ZG_PLAN_EAGER has none.
    if (!(flags & ZG_PLAN_EAGER) && hipStreamCreateWithFlags(&p->own_stream, hipStreamNonBlocking) != hipSuccess)
        return bail(fail(ZG_EHIP, "hipStreamCreateWithFlags failed"));
    // initial state: metadata, log, both bitmaps and the scan state zero (the id map needs no initial value:
    // an entry is only read for a vertex whose entry was written earlier in the same step)
    hipError_t e = hipMemsetAsync(p->ws + L.off_drmb, 0, sizeof(Drmb), st);
    if (e == hipSuccess) e = hipMemsetAsync(p->ws + L.off_log, 0, (size_t)kLogCapacity * ZG_LOG_STRIDE * 4, st);
    if (init_scratch) {
        if (e == hipSuccess) e = hipMemsetAsync(p->ws + L.off_seen, 0, (size_t)L.bitmap_words * 4, st);
        if (e == hipSuccess) e = hipMemsetAsync(p->ws + L.off_bitmap[0], 0, L.bitmap_bytes[0], st);
        if (e == hipSuccess) e = hipMemsetAsync(p->ws + L.off_bitmap[1], 0, L.bitmap_bytes[1], st);
        if (e == hipSuccess) e = hipMemsetAsync(p->ws + L.off_status, 0, L.status_words * 8, st);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return bail(fail(ZG_EHIP, std::string("initialising the workspace: ") + hipGetErrorString(e)));
    *out = p;
    return ZG_OK;
}

int zg_plan(zg_plan_t **out, const zg_graph_t *g, const int32_t *fanouts, int32_t num_hops, int32_t batch,
            const zg_envelope *env, int32_t feat_dim, void *d_workspace, size_t workspace_bytes, void *stream)
{
    if (!out) return fail(ZG_EINVAL, "null handle pointer");
    *out = nullptr;
    if (!g || g->stats_only) return fail(ZG_ESTATE, "zg_plan needs a graph handle with device arrays");
    Layout L, Ls;
    int rc = compute_layout(g, fanouts, num_hops, batch, env, feat_dim, nullptr, &L, &Ls);
    if (rc != ZG_OK) return rc;
    if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) % kAlign) != 0)
        return fail(ZG_EINVAL, "workspace must be a 256-byte aligned device pointer");
    if (workspace_bytes < L.total) return fail(ZG_ENOMEM, "workspace smaller than zg_plan_query's workspace_bytes");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(d_workspace);
    const bool with_twin = (env->flags & (ZG_PLAN_SAFE_TWIN | ZG_PLAN_AUTO_FALLBACK)) != 0;
    zg_plan_t *p = nullptr;
    // with a twin both lay their scratch out in the same region, sized for the larger of the two.  The id maps coincide; everything
    // behind them has to be zero between steps, whichever layout reads it: each of the two clears the regions of its own.
    rc = make_plan_object(&p, g, L, env->flags, batch, ws, st, true);
    if (rc != ZG_OK) return rc;
    if (with_twin) {
        rc = make_plan_object(&p->twin, g, Ls, env->flags & ~(ZG_PLAN_SAFE_TWIN | ZG_PLAN_AUTO_FALLBACK), batch, ws, st, true);
        if (rc == ZG_OK) rc = build_graph(p);
        if (rc != ZG_OK) {
            zg_plan_destroy(p);
            return rc;
        }
    }
    *out = p;
    return ZG_OK;
}

// host-only wait until the device has published that `target` of the steps the host has enqueued are finished; false after `seconds`
static bool wait_answered(const zg_plan_t *p, uint32_t target, double seconds)
{
    const volatile uint32_t *done = &p->mailbox->answered;
    const auto t0 = std::chrono::steady_clock::now();
    uint32_t polls = 0;
    while ((int32_t)(*done - target) < 0) {
        std::this_thread::yield();
        if ((++polls & 1023u) == 0 && std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() > seconds) return false;
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    return true;
}

constexpr double kHostWaitSeconds = 30.0;

int zg_plan_destroy(zg_plan_t *p)
{
    if (!p) return ZG_OK;
    // a step still in flight reads the mailbox and the captured graph: wait for this plan's own last step - its
    // completion counter first (host memory only), then the stream it was issued on, so that the launch has
    // retired as a whole.  Other plans' streams are not waited for, unless a recorded step may be in flight: where its
    // replays went the plan does not know.
    if (p->mailbox && (p->stepped || p->recorded)) {
        const bool done = !p->recorded && wait_answered(p, p->issued, kHostWaitSeconds);
        if (!done || hipStreamSynchronize(p->last_stream) != hipSuccess) {
            int device = p->device;
            (void)hipGetDevice(&device);
            (void)hipSetDevice(p->device);
            (void)hipDeviceSynchronize();
            (void)hipSetDevice(device);
        }
        (void)hipGetLastError();
    }
    if (p->twin) zg_plan_destroy(p->twin);
    drop_graph(p);
    if (p->own_stream) (void)hipStreamDestroy(p->own_stream);
    if (p->mailbox) (void)hipHostFree(p->mailbox);
    delete p;
    return ZG_OK;
}

int zg_plan_bind_features(zg_plan_t *p, const float *d_feat, int64_t ld)
{
    if (!p) return fail(ZG_EINVAL, "null plan");
    if (p->lay.feat_dim <= 0) return fail(ZG_ESTATE, "plan was made with feat_dim = 0");
    if (!d_feat || ld < p->lay.feat_dim) return fail(ZG_EINVAL, "null feature table or ld < feat_dim");
    p->d_feat = d_feat;
    p->ld_feat = ld;
    int rc = p->twin ? zg_plan_bind_features(p->twin, d_feat, ld) : ZG_OK; // first: the plan's graph may hold the twin's kernels
    if (rc == ZG_OK) rc = build_graph(p);
    return rc;
}

int zg_plan_outputs(const zg_plan_t *p, zg_outputs *o)
{
    if (!p || !o) return fail(ZG_EINVAL, "null argument");
    std::memset(o, 0, sizeof(*o));
    const Layout &L = p->lay;
    o->num_hops = L.num_hops;
    o->feat_dim = L.feat_dim;
    o->d_n = p->drmb()->n;
    o->d_E = p->drmb()->E;
    o->d_n_exact = p->drmb()->n_exact;
    o->d_flags = &p->drmb()->flags;
    o->d_S = p->S();
    for (int h = 0; h < L.num_hops; ++h) {
        o->d_row_ptr[h] = p->row_ptr(h);
        o->d_nbr_gid[h] = p->nbr(h);
        o->d_col[h] = p->col(h);
        o->edge_cap[h] = L.edge_cap[h];
    }
    for (int h = 0; h <= L.num_hops; ++h) o->node_cap[h] = L.node_cap[h];
    o->d_X = p->X();
    o->ldx = L.ld_out;
    o->d_agg = p->agg();
    o->ld_agg = L.ld_out;
    o->d_log = p->log();
    o->log_capacity = kLogCapacity;
    o->d_epoch = &p->drmb()->epoch;
    o->x_row_cap = L.x_rows;
    o->d_active = &p->drmb()->active;
    o->x_one_pass = x_written_by_aggregation(p) ? 1 : 0;
    return ZG_OK;
}

// zg_step and zg_step_timed.  The step's launches go into the stream one by one, the inputs with the first of them: the next step's first kernel
// starts when this one's last has ended, where the replay of a captured graph leaves the stream idle for 8 us, it reads its inputs from nowhere, and
// a launch costs the host 1.5 to 2 us where a replay costs it 15 to 25.  us per step replayed / launched, one plan: two hops of 717 edges 23.8 / 18.6, 2.4 M
// vertices, three hops and 250 k edges 113 / 108, two hops and 102 k edges 61.2 / 57.1, 110 M vertices 270 / 266; four plans on four streams, 64 seeds each: 26.6 / 7.1.
// A step with its twin's launches behind it (ZG_PLAN_AUTO_FALLBACK) is replayed: twice the launches gain little (107.4 / 104.1, the
// host 30 / 35), and that it is one graph launch is part of its contract.  (The mailbox slot is filled for every step: a step
// that is replayed may follow one that is not.)
static int issue_step(zg_plan_t *p, const int32_t *d_seeds, uint64_t rng_key, void *stream, StepProbe *probe)
{
    if (!p || !d_seeds) return fail(ZG_EINVAL, "null argument");
    if (p->broken) return fail(ZG_ESTATE, "an earlier step of this plan was enqueued in part: its scratch state is undefined");
    Queue q{static_cast<hipStream_t>(stream)};
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (q.st) ZG_HIP(hipStreamIsCapturing(q.st, &capture));
    q.recorded = capture != hipStreamCaptureStatusNone;
    const StepInputs in{d_seeds, rng_key};
    if (q.recorded) { // it runs, and counts as a step, when the caller replays it
        // (a replay would be a step that the host has filled no mailbox slot for, and every later one would read another step's)
        if (replays_graph(p)) return fail(ZG_ESTATE, "a step of a plan with ZG_PLAN_AUTO_FALLBACK cannot be recorded");
        const int rc = enqueue_step(p, q, in, probe);
        p->recorded = p->recorded || q.launched > 0;
        return rc;
    }
    // back-pressure without touching the device: wait (host only) while every mailbox slot is taken by a
    // step that has not finished yet
    if ((uint32_t)(p->issued - p->mailbox->answered) >= (uint32_t)kMailboxSlots - 1u &&
        !wait_answered(p, p->issued - ((uint32_t)kMailboxSlots - 2u), kHostWaitSeconds))
        return fail(ZG_ESTATE, "the device finished no step of this plan for 30 s while 255 are queued; nothing was enqueued");
    if (!probe && replays_graph(p) && !p->graph_exec) return fail(ZG_ESTATE, "plan has no captured graph");
    const uint32_t slot = p->issued % kMailboxSlots;
    p->mailbox->slot[slot].seeds = reinterpret_cast<unsigned long long>(d_seeds);
    p->mailbox->slot[slot].key = rng_key;
    std::atomic_thread_fence(std::memory_order_seq_cst);
    if (!probe && replays_graph(p)) {
        ZG_HIP(hipGraphLaunch(p->graph_exec, q.st));
    } else if (const int rc = enqueue_step(p, q, in, probe)) {
        if (q.launched > 0) { // (else nothing was enqueued: the slot is free again)
            p->broken = true;
            p->last_stream = q.st;
            p->stepped = true;
        }
        return rc;
    }
    // only now may an earlier step copy the slot ahead of time: a slot whose launch failed is filled again later
    p->issued += 1;
    reinterpret_cast<std::atomic<uint32_t> *>(&p->mailbox->issued)->store(p->issued, std::memory_order_release);
    p->last_stream = q.st;
    p->stepped = true;
    return ZG_OK;
}

int zg_step(zg_plan_t *p, const int32_t *d_seeds, uint64_t rng_key, void *stream)
{
    return issue_step(p, d_seeds, rng_key, stream, nullptr);
}

int zg_step_timed(zg_plan_t *p, const int32_t *d_seeds, uint64_t rng_key, void *stream, void *event_before, void *event_after)
{
    if (!event_before || !event_after) return fail(ZG_EINVAL, "null argument");
    if (p && !(p->d_feat && p->lay.feat_dim > 0)) return fail(ZG_ESTATE, "no feature table bound: the step has no aggregation launch");
    StepProbe probe{static_cast<hipEvent_t>(event_before), static_cast<hipEvent_t>(event_after), hipSuccess};
    const int rc = issue_step(p, d_seeds, rng_key, stream, &probe);
    if (rc == ZG_OK && probe.error != hipSuccess)
        return fail(ZG_EHIP, std::string("hipEventRecord: ") + hipGetErrorString(probe.error) + " (the step itself is enqueued)");
    return rc;
}

int zg_plan_replay_features(zg_plan_t *p, int32_t which, void *stream)
{
    if (!p) return fail(ZG_EINVAL, "null plan");
    if (!p->d_feat || p->lay.feat_dim <= 0) return fail(ZG_ESTATE, "no feature table is bound to the plan");
    if (which != 0 && which != 1) return fail(ZG_EINVAL, "which must be 0 (gather) or 1 (aggregation)");
    RowArgs gat, agg;
    step_feature_args(p, &gat, &agg);
    Queue q{static_cast<hipStream_t>(stream)};
    if (which == 0) return launch_gather(gat, relabel_args(p, 0, false), q);
    return launch_aggregate(agg, finish_args(p, false), q);
}

int zg_pilot_update(const zg_plan_t *p, int64_t *largest, void *stream)
{
    if (!p || !largest) return fail(ZG_EINVAL, "null argument");
    uint32_t n_exact[ZG_MAX_HOPS + 1];
    hipStream_t st = static_cast<hipStream_t>(stream);
    ZG_HIP(hipMemcpyAsync(n_exact, p->drmb()->n_exact, sizeof(n_exact), hipMemcpyDeviceToHost, st));
    ZG_HIP(hipStreamSynchronize(st));
    for (int h = 0; h <= p->lay.num_hops; ++h) largest[h] = std::max<int64_t>(largest[h], (int64_t)n_exact[h]);
    return ZG_OK;
}

#ifndef ZG_BUILD_ID
#define ZG_BUILD_ID "unknown"
#endif
const char *zg_build_id(void) { return ZG_BUILD_ID; }

int zg_calibration_copy(const void *d_src, void *d_dst, size_t bytes, void *stream)
{
    if (!d_src || !d_dst || bytes == 0 || (bytes & 15u) || (reinterpret_cast<uintptr_t>(d_src) & 15u) ||
        (reinterpret_cast<uintptr_t>(d_dst) & 15u))
        return fail(ZG_EINVAL, "zg_calibration_copy: pointers and size must be non-null multiples of 16");
    const size_t n = bytes / 16;
    const unsigned grid = (unsigned)std::min<size_t>((n + kBlock - 1) / kBlock, 256u * 64u);
    hipLaunchKernelGGL(k_calibrate_copy, dim3(grid), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint4 *>(d_src), static_cast<uint4 *>(d_dst), n);
    ZG_HIP(hipGetLastError());
    return ZG_OK;
}

int zg_envelope_model_graph(const zg_graph_t *g, const int32_t *fanouts, int32_t num_hops, int32_t batch, int32_t with_replacement,
                            const float *d_seed_prob, void *d_temp, size_t temp_bytes, void *stream, double *mean, double *sigma)
{
    if (!g || !fanouts || !mean || !sigma || !d_temp) return fail(ZG_EINVAL, "null argument");
    if (g->stats_only) return fail(ZG_ESTATE, "the graph-aware model needs a graph handle with device arrays");
    if (num_hops < 1 || num_hops > ZG_MAX_HOPS) return fail(ZG_EINVAL, "num_hops must be in 1..ZG_MAX_HOPS");
    if (batch < 1 || batch > g->num_nodes) return fail(ZG_EINVAL, "batch must be in 1..num_nodes");
    for (int h = 0; h < num_hops; ++h)
        if (fanouts[h] < 1 || fanouts[h] > ZG_MAX_FANOUT) return fail(ZG_EINVAL, "fanout must be in 1..ZG_MAX_FANOUT");
    const int64_t n = g->num_nodes;
    const size_t need = (size_t)n * 12 + 2 * kAlign + 64;
    if ((reinterpret_cast<uintptr_t>(d_temp) % kAlign) != 0 || temp_bytes < need)
        return fail(ZG_EINVAL, "temporary buffer must be 256-byte aligned and hold 12 bytes per vertex plus 576");
    int device = -1;
    ZG_HIP(hipGetDevice(&device));
    if (device != g->device) return fail(ZG_ESTATE, "current device differs from the graph's device");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(d_temp);
    unsigned long long *ell = reinterpret_cast<unsigned long long *>(base);
    size_t at = (size_t)n * 8;
    at = (at + kAlign - 1) / kAlign * kAlign;
    float *q = reinterpret_cast<float *>(base + at);
    at += (size_t)n * 4;
    at = (at + kAlign - 1) / kAlign * kAlign;
    unsigned long long *sums = reinterpret_cast<unsigned long long *>(base + at); // q and q (1 - q) of a hop, the next one's work; the first one's
    const ModelBins bins = model_bins(g, d_temp, at + 64, temp_bytes);
    // Which hops go by bins: those where the atomics would take longer.  With seeds given, a hop's terms may come from few of the edges:
    // the first hop's of a training set, all hops' of a handful of seeds.  A hop's work is counted by the update before it and known with
    // that one's sums; a probability never falls, so once by bins, always.  The first hop's is known to the device alone: it is
    // enqueued as if it was little, behind a gate; where it is not, nothing has happened but a look from the host.
    const int64_t all = g->num_edges + kModelRowWork * std::min(n, g->num_edges);
    auto by_bins = [&](int h, uint64_t work) { return bins.bins && work >= (uint64_t)model_bins_work(bins, num_hops - h); };
    bool binned = by_bins(0, (uint64_t)all), placed = false;
    ModelHop hop;
    std::memset(&hop, 0, sizeof(hop));
    hop.q = q;
    hop.ell = ell;
    hop.sums = sums;
    hop.replace = with_replacement;
    if (binned && d_seed_prob) {
        hop.rows.off = g->d_offsets;
        hop.rows.wide = g->offsets_dtype == ZG_I64;
        hop.gate.work = &sums[3];
        hop.gate.below = (uint64_t)model_bins_work(bins, num_hops);
        binned = false;
    }
    auto place_edges = [&]() {
        if (placed) return;
        placed = true;
        if (g->offsets_dtype == ZG_I64)
            enqueue_model_places<int64_t>(g, bins, st);
        else
            enqueue_model_places<int32_t>(g, bins, st);
    };
    auto clear_sums = [&]() { hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, reinterpret_cast<uint32_t *>(sums), 0u, (size_t)8); };
    if (binned) place_edges(); // (the longest launches first: the host is ahead of the device from here on)
    clear_sums();
    enqueue_model_init(g, q, ell, d_seed_prob, batch, hop.rows, &sums[3], st);
    ZG_HIP(hipGetLastError());
    mean[0] = (double)batch;
    sigma[0] = 0.0;
    int h = 0;
    while (h < num_hops && !binned) {
        hop.fanout = fanouts[h];
        if (h + 1 == num_hops) hop.rows.off = nullptr;
        enqueue_model_hop(g, bins, hop, st);
        ZG_HIP(hipGetLastError());
        unsigned long long host[4] = {0, 0, 0, 0};
        ZG_HIP(hipMemcpyAsync(host, sums, sizeof(host), hipMemcpyDeviceToHost, st));
        ZG_HIP(hipStreamSynchronize(st));
        const bool gated = hop.gate.work != nullptr;
        hop.gate.work = nullptr;
        if (gated && host[3] >= hop.gate.below) { // the gate was closed
            binned = true;
            continue;
        }
        mean[h + 1] = (double)host[0] / kFix;
        sigma[h + 1] = std::sqrt((double)host[1] / kFix);
        if (++h == num_hops) break;
        binned = hop.rows.off && by_bins(h, host[2]);
        clear_sums();
    }
    if (h < num_hops) { // the rest by bins, with nothing left to decide: one look at the end
        place_edges();
        hop.binned = true;
        hop.rows.off = nullptr;
        const int first = h;
        for (; h < num_hops; ++h) {
            hop.fanout = fanouts[h];
            hop.sums = bins.sums + 2 * h;
            enqueue_model_hop(g, bins, hop, st);
        }
        ZG_HIP(hipGetLastError());
        unsigned long long host[2 * ZG_MAX_HOPS];
        ZG_HIP(hipMemcpyAsync(host, bins.sums, sizeof(host), hipMemcpyDeviceToHost, st));
        ZG_HIP(hipStreamSynchronize(st));
        for (int i = first; i < num_hops; ++i) {
            mean[i + 1] = (double)host[2 * i] / kFix;
            sigma[i + 1] = std::sqrt((double)host[2 * i + 1] / kFix);
        }
    }
    return ZG_OK;
}

// device address of this GPU's copy of `scratch`, looked up once per device with that device current
static int static_scratch(int device, unsigned char **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static unsigned char *ptr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return fail(ZG_EINVAL, "device index out of range");
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[device]) {
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(zg::scratch));
        if (e != hipSuccess || !p) return fail(ZG_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        ptr[device] = static_cast<unsigned char *>(p);
    }
    *out = ptr[device];
    return ZG_OK;
}

int zg_envelope_model_graph_static(const zg_graph_t *g, const int32_t *fanouts, int32_t num_hops, int32_t batch,
                                   int32_t with_replacement, const float *d_seed_prob, void *stream, double *d_mean_sigma)
{
    if (!g || !fanouts || !d_mean_sigma) return fail(ZG_EINVAL, "null argument");
    if (g->stats_only) return fail(ZG_ESTATE, "the graph-aware model needs a graph handle with device arrays");
    if (num_hops < 1 || num_hops > ZG_MAX_HOPS) return fail(ZG_EINVAL, "num_hops must be in 1..ZG_MAX_HOPS");
    if (batch < 1 || batch > g->num_nodes) return fail(ZG_EINVAL, "batch must be in 1..num_nodes");
    for (int h = 0; h < num_hops; ++h)
        if (fanouts[h] < 1 || fanouts[h] > ZG_MAX_FANOUT) return fail(ZG_EINVAL, "fanout must be in 1..ZG_MAX_FANOUT");
    const int64_t n = g->num_nodes;
    if (n > (int64_t)ZG_STATIC_MODEL_MAX_NODES)
        return fail(ZG_EINVAL, "zg_envelope_model_graph_static: the graph has more vertices than ZG_STATIC_MODEL_MAX_NODES, the "
                               "capacity of the library's static scratch; use zg_envelope_model_graph with a caller buffer");
    if ((reinterpret_cast<uintptr_t>(d_mean_sigma) & 7u) != 0) return fail(ZG_EINVAL, "d_mean_sigma must be 8-byte aligned");
    int device = -1;
    ZG_HIP(hipGetDevice(&device));
    if (device != g->device) return fail(ZG_ESTATE, "current device differs from the graph's device");
    unsigned char *base = nullptr;
    int rc = static_scratch(device, &base);
    if (rc != ZG_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned long long *ell = reinterpret_cast<unsigned long long *>(base);
    float *q = reinterpret_cast<float *>(base + kStaticEllBytes);
    unsigned long long *sums = reinterpret_cast<unsigned long long *>(base + kStaticEllBytes + kStaticQBytes);
    ModelBins bins; // (no room for any)
    std::memset(&bins, 0, sizeof(bins));
    ModelHop hop;
    std::memset(&hop, 0, sizeof(hop));
    hop.q = q;
    hop.ell = ell;
    hop.replace = with_replacement;
    // the array keeps the last call's contents: the per-hop sums restart at zero here (a fill kernel, not a memset
    // node, so that the sequence may be captured), q and ell are overwritten for the first n vertices by the first kernel
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, reinterpret_cast<uint32_t *>(sums), 0u, (size_t)(4 * ZG_MAX_HOPS));
    enqueue_model_init(g, q, ell, d_seed_prob, batch, hop.rows, nullptr, st);
    ZG_HIP(hipGetLastError());
    for (int h = 0; h < num_hops; ++h) {
        hop.sums = sums + 2 * h;
        hop.fanout = fanouts[h];
        enqueue_model_hop(g, bins, hop, st);
        ZG_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_model_finish, dim3(1), dim3(64), 0, st, sums, num_hops, batch, d_mean_sigma);
    ZG_HIP(hipGetLastError());
    return ZG_OK;
}

int zg_step_safe(zg_plan_t *p, const int32_t *d_seeds, uint64_t rng_key, void *stream)
{
    if (!p) return fail(ZG_EINVAL, "null plan");
    if (!p->twin) return fail(ZG_ESTATE, "plan was made without ZG_PLAN_SAFE_TWIN");
    if (p->flags & ZG_PLAN_AUTO_FALLBACK)
        return fail(ZG_ESTATE, "with ZG_PLAN_AUTO_FALLBACK the twin runs inside zg_step, on the device's own decision");
    return zg_step(p->twin, d_seeds, rng_key, stream);
}

int zg_plan_outputs_safe(const zg_plan_t *p, zg_outputs *out)
{
    if (!p) return fail(ZG_EINVAL, "null plan");
    if (!p->twin) return fail(ZG_ESTATE, "plan was made without ZG_PLAN_SAFE_TWIN");
    return zg_plan_outputs(p->twin, out);
}

int zg_step_status(const zg_plan_t *p, uint32_t *steps_completed, uint32_t *last_flags)
{
    if (!p || !steps_completed || !last_flags) return fail(ZG_EINVAL, "null argument");
    const volatile Mailbox *m = p->mailbox;
    const uint32_t done = m->completed;
    std::atomic_thread_fence(std::memory_order_acquire);
    *steps_completed = done;
    *last_flags = done ? m->status[(done - 1) % kMailboxSlots] : 0u;
    return ZG_OK;
}

int zg_gather(zg_plan_t *p, const float *d_feat, int64_t ld, int32_t dim, float *d_out, int64_t ld_out, void *stream)
{
    if (!p || !d_feat || !d_out) return fail(ZG_EINVAL, "null argument");
    if (dim < 1 || dim > 32768 || ld < dim || ld_out < dim) return fail(ZG_EINVAL, "dim outside 1..32768 or a row stride < dim");
    const RowArgs gat = gather_args(p, d_feat, ld, dim, d_out, ld_out, p->lay.num_hops);
    Queue q{static_cast<hipStream_t>(stream)};
    return launch_gather(gat, relabel_args(p, 0, false), q);
}

int zg_aggregate_mean(zg_plan_t *p, int32_t hop, const float *d_in, int64_t ld_in, int32_t dim, float *d_out, int64_t ld_out,
                      void *stream)
{
    if (!p || !d_in || !d_out) return fail(ZG_EINVAL, "null argument");
    if (hop < 0 || hop >= p->lay.num_hops) return fail(ZG_EINVAL, "hop out of range");
    if (dim < 1 || dim > 32768 || ld_in < dim || ld_out < dim) return fail(ZG_EINVAL, "dim outside 1..32768 or a row stride < dim");
    const RowArgs agg = aggregate_args(p, hop, d_in, ld_in, dim, d_out, ld_out, false);
    Queue q{static_cast<hipStream_t>(stream)};
    return launch_aggregate(agg, finish_args(p, false), q);
}

int zg_overflow_flag(const zg_plan_t *p, const uint32_t **d_flag)
{
    if (!p || !d_flag) return fail(ZG_EINVAL, "null argument");
    *d_flag = &p->drmb()->flags;
    return ZG_OK;
}

int zg_overflow_clear(zg_plan_t *p, void *stream)
{
    if (!p) return fail(ZG_EINVAL, "null plan");
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), &p->drmb()->flags, 0u, (size_t)1);
    ZG_HIP(hipGetLastError());
    return ZG_OK;
}

} // extern "C"
