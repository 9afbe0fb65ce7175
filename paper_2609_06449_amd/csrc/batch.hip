// Batched form: many independent transforms of power-of-two sizes, all inside
// ONE kernel launch: in one workgroup up to 2^14 items, in two column passes
// above (tile.h; the single plans' direct form, whose bits it gives).
//
// Work is cut into tasks: up to 2^13 items of whole transforms of one size
// of at most 2^13 items, a whole transform of 2^14 items, or, for larger
// ones, one tile of the first or of the second column pass of one transform
// (2^14 items, 2^13 from a shared queue; "jobs" are the (transform, pass)
// pairs).  A batch of the first two kinds alone is a plain launch of one
// workgroup per task.  Otherwise the launch is persistent: a resident workgroup
// claims the next task number from an atomic ticket counter.  A pass-B task waits until every tile of its transform's pass A is done, on a
// per-job completion counter: the producer writes those tiles, waits for the
// stores to complete and then increments the counter; the consumer reads the
// counter and takes a device-scope acquire fence (which also drops stale
// cache lines) before touching the data.
//
// Forward progress: tickets are claimed in increasing order by workgroups
// that are already running, and a task only waits for jobs whose tasks all
// have smaller tickets.  The smallest unfinished ticket therefore never
// waits on anything unfinished, so every wait ends; each wait also gives up
// after a bounded number of polls and counts the event, so no wave can spin
// forever.  The schedule interleaves jobs so that a dependent job is usually
// emitted a couple of grid-widths of tiles after the job it waits for.
//
// The last workgroup to leave resets the ticket and completion counters, so
// the launch can be replayed (e.g. from a captured graph) without any memset.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <fstream>
#include <map>
#include <new>
#include <numeric>
#include <sstream>
#include <string>
#include <vector>

#include "paco.h"
#include "tile.h"

namespace paco {
namespace {

constexpr int kBT = 512;             // threads per workgroup of the persistent kernel
constexpr int kBatchMinLog2 = 2;     // N >= 4 (N1, N2 >= 2)
constexpr int kBatchMaxLog2 = 20;    // pass lengths <= 2^10
constexpr int kChipMaxLog2 = kDirectChipLog2;  // whole transform inside one workgroup
constexpr int kPassMin = 7, kPassMax = kBatchPassMax;
constexpr uint32_t kSpinLimit = 1u << 22;
// s_waitcnt operand that waits for vmcnt = 0 only (gfx9 encoding: vmcnt in
// bits 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima)
constexpr int kWaitStores = 0x0F70;
// s_getreg operand of the XCC_ID hardware register (id 20), bits 3:0: the
// XCD the reading wave runs on
constexpr int kHwRegXccId = 20 | (0 << 6) | ((4 - 1) << 11);
constexpr int kMaxQueues = 16;
constexpr int kTicketStride = 64;  // counters 256 bytes apart

enum : int32_t { kSmall = 0, kOne = 1, kPassA = 2, kPassB = 3 };

struct alignas(8) BatchJob {
    int64_t base;            // first item of the transform in in / out / workspace; kSmall: first entry of members
    int32_t kind;
    int32_t l1, l2;          // the passes' lengths 2^l1 (A), 2^l2 (B); kSmall: 2^l1 points
    int32_t count;           // kSmall: transforms of the task
    int32_t dep, dep_tiles;  // job this one waits for (-1: none) and its tile count
    int32_t ntiles;          // tasks of this job
    int32_t tab;             // table set of the transform size (kOne, kPassB)
    int32_t signal;          // 1: a later job waits for this one
    int32_t pad[3];
};

static_assert(sizeof(BatchJob) == 56, "job layout");

// One task: the tile number and a copy of its job (one 64-byte scalar load).
struct BatchTask {
    BatchJob J;
    uint32_t job, tile;
};

static_assert(sizeof(BatchTask) == 64, "task layout");

struct BatchArgs {
    const float2 *in;
    float2 *out;
    float2 *ws;
    const BatchTask *tasks;
    const BatchJob *jobs;
    const TopRoots *tabs;
    const int64_t *members;  // first items of the small transforms, task by task
    const float2 *stw;
    int32_t stw_off[kStageMaxLog2 + 1];
    uint32_t njobs;
    uint32_t nq;           // work queues: one per XCD, or one shared queue
    const uint32_t *qbeg;  // tasks of queue q: [qbeg[q], qbeg[q + 1])
    uint32_t *tickets;     // one counter per queue, kTicketStride apart
    uint32_t *exits, *done, *errors;
    uint32_t spin_limit;   // polls before a completion wait gives up (kSpinLimit)
};

// The thread id goes through an empty asm in every variant of a task: the
// compiler then hoists no variant's per-thread address arithmetic out of it
// (kept live across the others, it spilled).
__device__ __forceinline__ int own(int tid) { return int(opaque(uint32_t(tid))); }

constexpr int kLogBT = 9;      // the persistent kernel's threads
static_assert(kBT == 1 << kLogBT, "threads per workgroup");
// Batches without a transform of two passes need no work queue: a plain
// launch of one workgroup per task (batch_small_kernel), 256 threads and four
// workgroups per CU up to 2^12 items per transform, else 512 threads.
// 8192 transforms of 2^6..2^12: 38 us, through the queue 59, and 162 with one
// transform per workgroup and three phases through L2 (a copy takes 29).
constexpr int kLogST = 8, kShortMaxLog2 = 12;

constexpr int batch_lds()
{
    int m = tile_lds(13, 1, 2);  // kOne
    for (int l = kBatchMinLog2; l <= 13; ++l) m = m < tile_lds(l, small_lt(l, kLogBT), 1) ? tile_lds(l, small_lt(l, kLogBT), 1) : m;
    for (int l = kPassMin; l <= kPassMax; ++l) m = m < tile_lds(l, pass_lt(l, false), 2) ? tile_lds(l, pass_lt(l, false), 2) : m;
    return m;
}
static_assert(2 * (batch_lds() * 8 + 16) <= 160 * 1024, "two workgroups per CU");

constexpr int plain_lds(int lw)
{
    if (lw == kLogBT) return batch_lds();
    int m = 0;
    for (int l = kBatchMinLog2; l <= kShortMaxLog2; ++l)
        m = m < tile_lds(l, small_lt(l, lw), 1) ? tile_lds(l, small_lt(l, lw), 1) : m;
    return m;
}
static_assert(4 * plain_lds(kLogST) * 8 <= 160 * 1024, "four workgroups per CU");

template <int L, int LW>
__device__ __forceinline__ void run_small_len(const BatchArgs &A, const BatchJob &J, float2 *smem, int tid)
{
    static_assert(tile_threads(L, small_lt(L, LW), 1) == 1 << LW, "tile geometry");
    const int64_t *m = A.members + J.base;
    const int n = J.count;
    chip_tile<L, small_lt(L, LW)>(A.in, A.out, [&](int t) { return t < n ? m[t] : int64_t(-1); }, A.stw + A.stw_off[L],
                                  smem, own(tid), false, 0.f);
}

template <int LW>
__device__ __forceinline__ void run_small(const BatchArgs &A, const BatchJob &J, float2 *smem, int tid)
{
    switch (J.l1) {
    case 2: run_small_len<2, LW>(A, J, smem, tid); break;
    case 3: run_small_len<3, LW>(A, J, smem, tid); break;
    case 4: run_small_len<4, LW>(A, J, smem, tid); break;
    case 5: run_small_len<5, LW>(A, J, smem, tid); break;
    case 6: run_small_len<6, LW>(A, J, smem, tid); break;
    case 7: run_small_len<7, LW>(A, J, smem, tid); break;
    case 8: run_small_len<8, LW>(A, J, smem, tid); break;
    case 9: run_small_len<9, LW>(A, J, smem, tid); break;
    case 10: run_small_len<10, LW>(A, J, smem, tid); break;
    case 11: run_small_len<11, LW>(A, J, smem, tid); break;
    case 12: run_small_len<12, LW>(A, J, smem, tid); break;
    default:
        if constexpr (LW >= kLogBT) run_small_len<13, LW>(A, J, smem, tid);
        break;
    }
}

__device__ __forceinline__ void run_one(const BatchArgs &A, const BatchJob &J, float2 *smem, int tid)
{
    const TopRoots T = A.tabs[J.tab];
    chip14_tile(A.in + J.base, A.out + J.base, A.stw + A.stw_off[13], T.hi, T.lo, smem, own(tid), false, 0.f);
}

// A batch of transforms of one workgroup: workgroup i runs task i.
template <int LW>
__global__ __launch_bounds__(1 << LW) void batch_small_kernel(BatchArgs A)
{
    __shared__ float2 smem[plain_lds(LW)];
    const BatchJob &J = A.jobs[blockIdx.x];
    if constexpr (LW >= kLogBT) {
        if (J.kind == kOne) {
            run_one(A, J, smem, threadIdx.x);
            return;
        }
    }
    run_small<LW>(A, J, smem, threadIdx.x);
}

template <int L, bool COH>
__device__ __forceinline__ void run_a_len(const BatchArgs &A, const BatchJob &J, uint32_t tile, float2 *smem, int tid)
{
    constexpr int LT = pass_lt(L, COH), H = COH ? 1 : 2;
    static_assert(tile_threads(L, LT, H) == kBT, "tile geometry");
    pass_a_tile<L, LT, H, COH>(A.in + J.base, A.ws + J.base, J.l2, pass_lt(J.l2, COH), tile << LT, A.stw + A.stw_off[L],
                               smem, own(tid), false);
}

template <int L, bool COH>
__device__ __forceinline__ void run_b_len(const BatchArgs &A, const BatchJob &J, uint32_t tile, float2 *smem, int tid)
{
    constexpr int LT = pass_lt(L, COH), H = COH ? 1 : 2;
    pass_b_tile<L, LT, H>(A.ws + J.base, A.out + J.base, J.l1, tile << LT, A.tabs[J.tab], A.stw + A.stw_off[L], smem,
                          own(tid), 0.f);
}

template <bool COH>
__device__ __forceinline__ void run_a(const BatchArgs &A, const BatchJob &J, uint32_t tile, float2 *smem, int tid)
{
    switch (J.l1) {
    case 7: run_a_len<7, COH>(A, J, tile, smem, tid); break;
    case 8: run_a_len<8, COH>(A, J, tile, smem, tid); break;
    case 9: run_a_len<9, COH>(A, J, tile, smem, tid); break;
    default: run_a_len<10, COH>(A, J, tile, smem, tid); break;
    }
}

template <bool COH>
__device__ __forceinline__ void run_b(const BatchArgs &A, const BatchJob &J, uint32_t tile, float2 *smem, int tid)
{
    switch (J.l2) {
    case 7: run_b_len<7, COH>(A, J, tile, smem, tid); break;
    case 8: run_b_len<8, COH>(A, J, tile, smem, tid); break;
    case 9: run_b_len<9, COH>(A, J, tile, smem, tid); break;
    default: run_b_len<10, COH>(A, J, tile, smem, tid); break;
    }
}

// Polls with relaxed loads (an acquire load also drops this XCD's cached
// lines, which would slow every other workgroup on it while one waits), then
// one device-scope acquire fence once the count is reached.
__device__ __forceinline__ void wait_for(const BatchArgs &A, int32_t dep, uint32_t need)
{
    uint32_t spins = 0;
    while (__hip_atomic_load(A.done + dep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
        __builtin_amdgcn_s_sleep(8);
        if (++spins >= A.spin_limit) {
            atomicAdd(A.errors, 1u);
            break;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// COH = false: one work queue per XCD.  A workgroup serves the queue of the
// XCD it runs on (read from the hardware), and every task of a transform sits
// in one queue, so producer and consumer tiles share that XCD's L2: ordinary
// stores, completed (vmcnt 0) before the counter moves, are what the
// consumer reads after its acquire fence (which drops stale L1 lines).
// COH = true: one queue shared by all XCDs; the tiles other tasks read are
// written with device-coherent stores instead.
template <bool COH>
__global__ __launch_bounds__(kBT) __attribute__((amdgpu_waves_per_eu(4))) void batch_kernel(BatchArgs A)
{
    __shared__ float2 smem[batch_lds()];
    __shared__ uint32_t s_ticket;
    __shared__ int s_last;
    const int tid = threadIdx.x;
    const uint32_t q = COH ? 0u : uint32_t(__builtin_amdgcn_s_getreg(kHwRegXccId)) % A.nq;
    uint32_t *ticket = A.tickets + q * kTicketStride;
    const uint32_t beg = A.qbeg[q], end = A.qbeg[q + 1];
    if (tid == 0) s_ticket = beg + atomicAdd(ticket, 1u);
    __syncthreads();
    uint32_t tk = __builtin_amdgcn_readfirstlane(s_ticket);
    for (;;) {
        if (tk >= end) break;
        const BatchTask &task = A.tasks[tk];  // (read where used: held in registers it spilled)
        const BatchJob &J = task.J;
        // the next ticket is claimed now and read after the task, so the
        // atomic's round trip overlaps the work
        uint32_t next = 0;
        if (tid == 0) next = beg + atomicAdd(ticket, 1u);
        if (J.dep >= 0) {
            if (tid == 0) wait_for(A, J.dep, uint32_t(J.dep_tiles));
            __syncthreads();
        }
        switch (J.kind) {
        case kPassA: run_a<COH>(A, J, task.tile, smem, tid); break;
        case kPassB: run_b<COH>(A, J, task.tile, smem, tid); break;
        case kOne: run_one(A, J, smem, tid); break;
        default: run_small<kLogBT>(A, J, smem, tid); break;
        }
        // Completion: once every wave has seen its stores complete (vmcnt 0)
        // a relaxed device-scope increment publishes the tile (the ordering a
        // release gives, without writing back the whole L2 of the XCD).
        if (J.signal) __builtin_amdgcn_s_waitcnt(kWaitStores);
        if (tid == 0) s_ticket = next;
        __syncthreads();  // LDS free for the next task; s_ticket written
        if (J.signal && tid == 0) __hip_atomic_fetch_add(A.done + task.job, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tk = __builtin_amdgcn_readfirstlane(s_ticket);
        __syncthreads();  // every wave has read s_ticket before thread 0 writes it again
    }
    // Leaving: no order but "this workgroup's counter updates are performed
    // before its exit is counted" is needed, so a wait and a relaxed add (an
    // acquire-release add wrote back and dropped the XCD's L2 once per
    // workgroup: with 512 of them 36.6 us for 512 transforms of 2^13).
    if (tid == 0) {
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
        s_last = __hip_atomic_fetch_add(A.exits, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    }
    __syncthreads();
    if (s_last) {  // everyone else has left: rearm the counters for the next launch
        // a queue whose ticket never reached its length had tasks no
        // workgroup ran (no workgroup landed on its XCD): count them
        for (uint32_t j = tid; j < A.nq; j += kBT) {
            const uint32_t got = __hip_atomic_load(A.tickets + j * kTicketStride, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t len = A.qbeg[j + 1] - A.qbeg[j];
            if (got < len) atomicAdd(A.errors, len - got);
        }
        __syncthreads();  // every queue checked before its ticket is rearmed
        const auto clear = [](uint32_t *c) { __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        for (uint32_t j = tid; j < A.njobs; j += kBT) clear(A.done + j);
        for (uint32_t j = tid; j < A.nq; j += kBT) clear(A.tickets + j * kTicketStride);
        if (tid == 0) clear(A.exits);
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
struct SizePlan {
    int l1 = 0, l2 = 0, t = 1;
};

int ilog2_pow2(int64_t n)
{
    if (n < 1 || (n & (n - 1))) return -1;
    int l = 0;
    while ((int64_t(1) << l) < n) ++l;
    return l;
}

// Valid per-size plans, default first: balanced split, b = 2.  The plan of
// transforms of at most 2^14 items has no choice that matters (one workgroup
// runs all of it); of larger ones the split decides the lengths of the two
// passes.  b is reported and has no effect on the result or the time.
std::vector<SizePlan> candidates(int k)
{
    std::vector<SizePlan> out;
    const int mid = (k + 1) / 2;
    out.push_back({mid, k - mid, 1});
    for (int l = kPassMin; l <= kPassMax; ++l)
        if (l != mid && batch_split(l, k - l)) out.push_back({l, k - l, 1});
    return out;
}

}  // namespace
}  // namespace paco

using paco::BatchArgs;
using paco::BatchJob;
using paco::BatchTask;
using paco::SizePlan;

struct paco_batch_plan_s {
    int32_t count = 0;
    std::vector<int64_t> N, offset;
    std::map<int, SizePlan> plans;  // by log2 N
    int64_t total = 0;
    int device = 0;
    void *dev = nullptr;
    BatchArgs args{};
    int grid = 0;
    int64_t gap = 0;
    int nq = 1;        // work queues
    bool coh = false;  // one queue served by several XCDs: coherent stores
    int lw = 0;        // log2 threads of a plain launch (batch_small_kernel); 0: the persistent kernel
    paco_batch_options opt{};
    std::string desc;
};

namespace {

paco_status bfail(paco_status st, const std::string &msg)
{
    paco::set_last_error(msg);
    return st;
}

// (the runtime's last error is taken back: see hip_fail in plan.hip)
paco_status bhip(hipError_t e, const char *what, paco_status st = PACO_ERR_HIP)
{
    (void)hipGetLastError();
    return bfail(st, std::string(what) + ": " + hipGetErrorString(e));
}

const void *kernel_of(bool coh)
{
    return coh ? reinterpret_cast<const void *>(paco::batch_kernel<true>)
               : reinterpret_cast<const void *>(paco::batch_kernel<false>);
}

int resident_workgroups(bool coh)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const hipError_t e = coh ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, paco::batch_kernel<true>, paco::kBT, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, paco::batch_kernel<false>, paco::kBT, 0);
    if (e != hipSuccess) return 0;
    return cus * std::max(per, 1);
}

const void *small_kernel_of(int lw)
{
    return lw == paco::kLogST ? reinterpret_cast<const void *>(paco::batch_small_kernel<paco::kLogST>)
                              : reinterpret_cast<const void *>(paco::batch_small_kernel<paco::kLogBT>);
}

int resident_small(int lw)
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, small_kernel_of(lw), 1 << lw, 0) != hipSuccess)
        return 0;
    return cus * std::max(per, 1);
}

// Work queues: one per XCD of the device (the option PACO_BATCH_ONE_QUEUE
// forces one shared queue with device-coherent stores).
int queue_count(const paco_batch_options &opt)
{
    int dev = 0, nx = 0;
    if (opt.flags & PACO_BATCH_ONE_QUEUE) return 1;
    if (hipGetDevice(&dev) != hipSuccess) return 1;
    if (hipDeviceGetAttribute(&nx, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess) return 1;
    return (nx >= 1 && nx <= paco::kMaxQueues) ? nx : 1;
}

// Deals the transforms to the work queues, largest first onto the least loaded
// (returned queue by queue), and sets which kernel runs them (lw, nq, coh).
typedef std::vector<std::vector<int32_t>> Queues;
Queues deal_queues(paco_batch_plan_s *P)
{
    using namespace paco;
    int nx = queue_count(P->opt);
    int dev = 0, nxcd = 1;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&nxcd, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess)
        nxcd = 0;  // unknown: one shared, coherent queue
    std::vector<int32_t> order(P->count);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return P->N[a] > P->N[b]; });
    Queues qorder;
    const auto deal = [&](int n) {  // returns the largest queue's items
        std::vector<int64_t> load(n, 0);
        qorder.assign(n, {});
        for (int32_t i : order) {
            const int qi = int(std::min_element(load.begin(), load.end()) - load.begin());
            load[qi] += P->N[i];
            qorder[qi].push_back(i);
        }
        return *std::max_element(load.begin(), load.end());
    };
    // A queue per XCD keeps a transform's intermediate in that XCD's L2, but
    // a transform then runs on one XCD alone: where the fullest queue would
    // hold more than 1.5 times its share (a few large transforms), all XCDs
    // serve one queue.  Both sides, us from a queue per XCD / a shared one:
    //   times its share           2^16          2^18          2^20
    //   8    (1 transform)     81 / 21      101 / 22      112 / 29
    //   2.67 (3)               43 / 22       56 / 30       73 / 71
    //   2    (4)               23 / 23       33 / 32       69 / 83
    //   1.78 (9)               26 / 28       45 / 70      110 / 95
    //   1.6  (10)              26 / 29       48 / 74      113 / 122
    //   1.33 (12)              27 / 31       53 / 78      117 / 153
    //   1    (8)               25 / 26       38 / 67       87 / 97
    // 2^20 with 3000 of 2^6 .. 2^12 (1.85) 59 / 45, three of them (1.27) 65 / 50, 2^20
    // with 16 of 2^18 (1.6) 68 / 92.  Up to 1.5 the queues per XCD win on all but a
    // few of the lists, above 2 the shared one; between, neither does throughout,
    // and the line leaves it to the shared queue.
    const int kmax = ilog2_pow2(P->N[order[0]]);
    P->lw = kmax <= kShortMaxLog2 ? kLogST : kmax <= kChipMaxLog2 ? kLogBT : 0;
    if (P->lw) nx = 1;
    if (deal(nx) * nx > P->total + P->total / 2 && nx > 1) {
        nx = 1;
        deal(nx);
    }
    P->coh = nx == 1 && nxcd != 1;  // several XCDs serve one queue
    P->nq = nx;
    return qorder;
}

// Builds jobs, the task order and the device tables of a batch whose
// per-size plans are fixed and whose transforms are dealt (qorder).  Returns
// PACO_OK or an error with the detail set.
paco_status build_batch(paco_batch_plan_s *P, const Queues &qorder)
{
    using namespace paco;
    const int32_t count = P->count;
    // ---- per-size Phase II tables and the stage tables -----------------------
    std::vector<int> ks;
    for (auto &kv : P->plans) ks.push_back(kv.first);
    std::map<int, int> tab_of;
    std::vector<std::vector<float2>> his, los, cws;
    for (int k : ks) {
        if (k < kChipMaxLog2) continue;  // no table but the stages'
        tab_of[k] = int(his.size());
        std::vector<float2> hi, lo, cw;
        top_tables(k, hi, lo);
        if (k > kChipMaxLog2) {
            const int64_t n = int64_t(16) << P->plans[k].l1;
            cw.resize(size_t(n));
            for (int64_t i = 0; i < n; ++i) cw[i] = root_neg(i, n);
        }
        his.push_back(std::move(hi));
        los.push_back(std::move(lo));
        cws.push_back(std::move(cw));
    }
    std::vector<float2> stw;
    int64_t stw_off[kStageMaxLog2 + 1];
    if (!stage_tables(stw, stw_off)) return bfail(PACO_ERR_INVALID_ARG, "internal: stage twiddle layout mismatch");

    const int nx = P->nq, lw = P->lw ? P->lw : kLogBT;
    const int resident = P->lw ? resident_small(P->lw) : resident_workgroups(P->coh);
    if (resident <= 0) return bfail(PACO_ERR_HIP, "occupancy query failed");

    // ---- jobs ---------------------------------------------------------------
    std::vector<BatchJob> jobs;
    std::vector<int64_t> members;
    struct Chain { int32_t first; };  // pass-A job of a large transform (pass B = +1)
    std::vector<std::vector<Chain>> chains(nx);
    std::vector<std::vector<int32_t>> smalls(nx);
    for (int qi = 0; qi < nx; ++qi) {
        // items of a small task: a full tile, less where that would leave
        // workgroups of the queue without one
        int64_t small_items = 0;
        for (int32_t i : qorder[qi])
            if (ilog2_pow2(P->N[i]) < kChipMaxLog2) small_items += P->N[i];
        const int64_t share = small_items * nx / resident + 1;
        for (size_t o = 0; o < qorder[qi].size(); ++o) {
            const int32_t i = qorder[qi][o];
            const int k = ilog2_pow2(P->N[i]);
            const SizePlan &sp = P->plans[k];
            BatchJob J{};
            J.base = P->offset[i];
            J.l1 = sp.l1;
            J.l2 = sp.l2;
            J.dep = -1;
            J.ntiles = 1;
            if (k < kChipMaxLog2) {  // with the next transforms of its size
                const int64_t most = std::max<int64_t>(1, std::min<int64_t>(share >> k, int64_t(1) << small_lt(k, lw)));
                J.kind = kSmall;
                J.l1 = k;
                J.base = int64_t(members.size());
                while (o < qorder[qi].size() && P->N[qorder[qi][o]] == P->N[i] && J.count < most) {
                    members.push_back(P->offset[qorder[qi][o]]);
                    ++J.count;
                    ++o;
                }
                --o;
                smalls[qi].push_back(int32_t(jobs.size()));
                jobs.push_back(J);
                continue;
            }
            J.tab = tab_of[k];
            if (k == kChipMaxLog2) {
                J.kind = kOne;
                smalls[qi].push_back(int32_t(jobs.size()));
                jobs.push_back(J);
                continue;
            }
            const int32_t first = int32_t(jobs.size());
            BatchJob a = J, c = J;
            a.kind = kPassA;
            a.ntiles = 1 << (sp.l2 - pass_lt(sp.l1, P->coh));
            a.signal = 1;
            c.kind = kPassB;
            c.ntiles = 1 << (sp.l1 - pass_lt(sp.l2, P->coh));
            c.dep = first;
            c.dep_tiles = a.ntiles;
            jobs.push_back(a);
            jobs.push_back(c);
            chains[qi].push_back({first});
        }
    }

    // ---- launch geometry -----------------------------------------------------
    // per queue: a job's successor is emitted about `gap` tiles after it:
    // twice the workgroups that serve the queue, so that it rarely waits and
    // the intermediate is still near (batch of 4096 transforms 2^8..2^20 by
    // the gap in workgroups per queue: 0.5 4.71 ms, 1 4.26, 2 3.77, 4 4.17)
    P->gap = 2 * int64_t(resident) / nx;
    if (P->opt.flags & PACO_BATCH_SET_GAP) P->gap = P->opt.gap;

    // ---- task order, queue by queue ------------------------------------------
    std::vector<BatchTask> tasks;
    std::vector<uint32_t> qbeg;
    for (int qi = 0; qi < nx; ++qi) {
        qbeg.push_back(uint32_t(tasks.size()));
        const int64_t base = int64_t(tasks.size());
        std::deque<std::pair<int64_t, int32_t>> pending;  // (ready position, job)
        auto emit = [&](int32_t j) {
            for (int32_t t = 0; t < jobs[j].ntiles; ++t) tasks.push_back({jobs[j], uint32_t(j), uint32_t(t)});
            if (jobs[j].kind == kPassA)
                pending.push_back({int64_t(tasks.size()) - base + P->gap, j + 1});
        };
        auto pos = [&]() { return int64_t(tasks.size()) - base; };
        size_t next_small = 0;
        const std::vector<int32_t> &sm = smalls[qi];
        for (const Chain &ch : chains[qi]) {
            while (!pending.empty() && pending.front().first <= pos()) {
                const int32_t j = pending.front().second;
                pending.pop_front();
                emit(j);
            }
            emit(ch.first);
        }
        while (!pending.empty()) {
            if (pending.front().first > pos() && next_small < sm.size()) {
                emit(sm[next_small++]);
                continue;
            }
            const int32_t j = pending.front().second;
            pending.pop_front();
            emit(j);
        }
        while (next_small < sm.size()) emit(sm[next_small++]);
    }
    qbeg.push_back(uint32_t(tasks.size()));
    if (tasks.size() >= 0xffffffffull) return bfail(PACO_ERR_UNSUPPORTED, "too many tasks");

    // ---- one device allocation ----------------------------------------------
    struct Piece { const void *src; size_t bytes; size_t off; };
    std::vector<Piece> pieces;
    auto add = [&](const void *src, size_t bytes) {
        pieces.push_back({src, bytes, 0});
        return pieces.size() - 1;
    };
    const size_t i_stw = add(stw.data(), stw.size() * 8);
    std::vector<size_t> i_hi, i_lo, i_cw;
    for (size_t s = 0; s < his.size(); ++s) {
        i_hi.push_back(add(his[s].data(), his[s].size() * 8));
        i_lo.push_back(add(los[s].data(), los[s].size() * 8));
        i_cw.push_back(add(cws[s].data(), cws[s].size() * 8));
    }
    std::vector<TopRoots> tabs(his.size());
    const size_t i_tabs = add(nullptr, tabs.size() * sizeof(TopRoots));
    const size_t i_mem = add(members.data(), members.size() * 8);
    const size_t i_jobs = add(jobs.data(), jobs.size() * sizeof(BatchJob));
    const size_t i_tasks = add(tasks.data(), tasks.size() * sizeof(BatchTask));
    const size_t i_qbeg = add(qbeg.data(), qbeg.size() * 4);
    const size_t i_tick = add(nullptr, size_t(nx) * kTicketStride * 4);  // one 256-byte block per queue
    const size_t i_cnt = add(nullptr, 256 * 2);                          // exits, errors
    const size_t i_done = add(nullptr, jobs.size() * 4);
    size_t total = 0;
    for (auto &pc : pieces) {
        pc.off = total;
        total += (pc.bytes + 255) & ~size_t(255);
    }
    hipError_t e = hipMalloc(&P->dev, total);
    if (e != hipSuccess) {
        P->dev = nullptr;
        return bhip(e, "hipMalloc", PACO_ERR_ALLOC);
    }
    auto at = [&](size_t i) { return static_cast<unsigned char *>(P->dev) + pieces[i].off; };
    for (size_t s = 0; s < his.size(); ++s) {
        tabs[s].hi = reinterpret_cast<const float2 *>(at(i_hi[s]));
        tabs[s].lo = reinterpret_cast<const float2 *>(at(i_lo[s]));
        tabs[s].cw = reinterpret_cast<const float2 *>(at(i_cw[s]));
    }
    for (const auto &kt : tab_of) {
        tabs[kt.second].log2N = kt.first;
        tabs[kt.second].log2Lo = middle_log2lo(kt.first);
    }
    pieces[i_tabs].src = tabs.data();
    std::vector<unsigned char> staging(total, 0);  // counters start at zero
    for (auto &pc : pieces)
        if (pc.src) std::memcpy(staging.data() + pc.off, pc.src, pc.bytes);
    e = hipMemcpy(P->dev, staging.data(), total, hipMemcpyHostToDevice);
    if (e != hipSuccess) return bhip(e, "hipMemcpy");

    BatchArgs &A = P->args;
    A.tasks = reinterpret_cast<const BatchTask *>(at(i_tasks));
    A.jobs = reinterpret_cast<const BatchJob *>(at(i_jobs));
    A.tabs = reinterpret_cast<const TopRoots *>(at(i_tabs));
    A.members = reinterpret_cast<const int64_t *>(at(i_mem));
    A.stw = reinterpret_cast<const float2 *>(at(i_stw));
    for (int l = 0; l <= kStageMaxLog2; ++l) A.stw_off[l] = int32_t(stw_off[l]);
    A.njobs = uint32_t(jobs.size());
    A.nq = uint32_t(nx);
    A.qbeg = reinterpret_cast<const uint32_t *>(at(i_qbeg));
    A.tickets = reinterpret_cast<uint32_t *>(at(i_tick));
    A.exits = reinterpret_cast<uint32_t *>(at(i_cnt));
    A.errors = reinterpret_cast<uint32_t *>(at(i_cnt) + 256);
    // option: a tiny poll limit forces the give-up path from the host
    // (every wave still exits; results are then unspecified)
    A.spin_limit = P->opt.spin_limit ? P->opt.spin_limit : kSpinLimit;
    A.done = reinterpret_cast<uint32_t *>(at(i_done));
    // at least one workgroup per queue: workgroups are dealt to the XCDs in
    // turn, so every XCD's queue has a server (the exit check of the kernel
    // counts any queue left unserved anyway)
    P->grid = P->lw ? int(jobs.size())
                    : int(std::max<int64_t>(std::min<int64_t>(int64_t(resident), int64_t(tasks.size())), int64_t(nx)));

    char buf[256];
    std::snprintf(buf, sizeof buf,
                  "batch[%d transforms, %lld items, %zu jobs, %zu tasks, %d %s, grid %d x %d, lds %zu, gap %lld]",
                  count, (long long)P->total, jobs.size(), tasks.size(), nx,
                  P->lw ? "task list (one workgroup per task)"
                  : P->coh ? "shared queue (coherent stores)"
                           : "queues (one per XCD)",
                  P->grid, 1 << lw, size_t(paco::plain_lds(lw)) * 8,
                  (long long)P->gap);
    P->desc = buf;
    for (auto &kv : P->plans) {
        const SizePlan &sp = kv.second;
        std::snprintf(buf, sizeof buf, " 2^%d:%dx%d,b=%d%s", kv.first, 1 << sp.l1, 1 << sp.l2, 1 << sp.t,
                      kv.first <= kChipMaxLog2 ? "(wg)" : "");
        P->desc += buf;
    }
    if (const char *lg = std::getenv("PACO_LOG"))  // plan summary on stderr
        if (lg[0] == '1') std::fprintf(stderr, "paco batch plan: %s\n", P->desc.c_str());
    return PACO_OK;
}

hipError_t launch_batch(const paco_batch_plan_s *P, const void *in, void *out, void *ws, hipStream_t s)
{
    BatchArgs A = P->args;
    A.in = static_cast<const float2 *>(in);
    A.out = static_cast<float2 *>(out);
    A.ws = static_cast<float2 *>(ws);
    void *args[] = {&A};
    if (P->lw) return hipLaunchKernel(small_kernel_of(P->lw), dim3(unsigned(P->grid)), dim3(1u << P->lw), args, 0, s);
    return hipLaunchKernel(kernel_of(P->coh), dim3(unsigned(P->grid)), dim3(paco::kBT), args, 0, s);
}

void free_plan(paco_batch_plan_s *P)
{
    if (!P) return;
    if (P->dev) (void)hipFree(P->dev);
    delete P;
}

// ---- autotuner -----------------------------------------------------------------
// For every transform size of the batch, each candidate split runs a batch of
// copies of that size (about 2^24 items) through the persistent kernel; the
// fastest of three timed launches wins.  Where the batch runs from one shared
// queue (P->coh: a few large transforms, half-width tiles, coherent stores), so
// do the trials, with no more copies than the batch has of the size, and eight
// launches are timed together: nine transforms of 2^18 take 58 us as 1024 x 256
// and 70 as 512 x 512 there, 256 of them from a queue per XCD 381 and 389.
paco_status tune(const paco_batch_plan_s *P, std::map<int, SizePlan> &plans, const std::vector<int> &ks)
{
    bool choice = false;
    for (int k : ks) {
        const std::vector<SizePlan> cand = paco::candidates(k);
        plans[k] = cand.front();
        choice = choice || cand.size() > 1;
    }
    if (!choice) return PACO_OK;
    const int64_t items = int64_t(1) << 24;
    void *buf = nullptr;
    hipError_t e = hipMalloc(&buf, size_t(items) * 8 * 3);
    if (e != hipSuccess) return bhip(e, "tuning buffers", PACO_ERR_ALLOC);
    float2 *in = static_cast<float2 *>(buf), *out = in + items, *ws = out + items;
    hipStream_t s = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    paco_status st = PACO_OK;
    if ((e = hipMemset(buf, 0, size_t(items) * 8 * 3)) != hipSuccess || (e = hipStreamCreate(&s)) != hipSuccess ||
        (e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess) {
        st = bhip(e, "tuning set-up");
    }
    for (size_t ki = 0; st == PACO_OK && ki < ks.size(); ++ki) {
        const int k = ks[ki];
        int64_t copies = std::min<int64_t>(std::max<int64_t>(1, items >> k), 16384);
        if (P->coh) copies = std::min<int64_t>(copies, std::count(P->N.begin(), P->N.end(), int64_t(1) << k));
        const int launches = P->coh ? 8 : 1;
        float best = 1e30f;
        const std::vector<SizePlan> cand = paco::candidates(k);
        if (cand.size() == 1) continue;
        for (const SizePlan &sp : cand) {
            paco_batch_plan_s *T = new (std::nothrow) paco_batch_plan_s();
            if (!T) { st = bfail(PACO_ERR_ALLOC, "host allocation failed"); break; }
            T->count = int32_t(copies);
            for (int64_t i = 0; i < copies; ++i) {
                T->N.push_back(int64_t(1) << k);
                T->offset.push_back(i << k);
            }
            T->total = copies << k;
            T->plans[k] = sp;
            if (P->coh) T->opt.flags |= PACO_BATCH_ONE_QUEUE;
            st = build_batch(T, deal_queues(T));
            float ms = 1e30f;
            for (int rep = 0; st == PACO_OK && rep < 4; ++rep) {
                e = hipEventRecord(e0, s);
                for (int i = 0; e == hipSuccess && i < launches; ++i) e = launch_batch(T, in, out, ws, s);
                if (e != hipSuccess || (e = hipEventRecord(e1, s)) != hipSuccess ||
                    (e = hipEventSynchronize(e1)) != hipSuccess) {
                    st = bhip(e, "tuning launch");
                    break;
                }
                float t = 0.f;
                (void)hipEventElapsedTime(&t, e0, e1);
                if (rep > 0) ms = std::min(ms, t);  // the first launch warms up
            }
            free_plan(T);
            if (st != PACO_OK) break;
            if (ms < best) {
                best = ms;
                plans[k] = sp;
            }
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (s) (void)hipStreamDestroy(s);
    (void)hipFree(buf);
    return st;
}

// A cached plan is used if its split is one of the candidates' (any split of
// a transform of one workgroup) and its b is a base of both sides.
bool valid_plan(int k, const SizePlan &sp)
{
    if (sp.t != 1 && sp.t != 2 && sp.t != 4) return false;
    if (sp.l1 < 1 || sp.l2 < 1 || sp.l1 + sp.l2 != k || sp.l1 % sp.t || sp.l2 % sp.t) return false;
    if (k <= paco::kChipMaxLog2) return true;
    for (const SizePlan &c : paco::candidates(k))
        if (c.l1 == sp.l1) return true;
    return false;
}

// The device and the kernels a tuning cache was measured on: its entries are
// reused only on the same architecture and CU count, and only while format
// stands.  A change of the passes that the candidates are timed on takes a new
// number, also where the lines look the same (format 1: three phases per
// transform, whose timings say nothing about the two column passes; format 2:
// lines without the queue mode).
std::string cache_key()
{
    int dev = 0;
    hipDeviceProp_t prop{};
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return "unknown";
    std::string arch = prop.gcnArchName;
    for (char &ch : arch)
        if (ch == ' ') ch = '_';
    return arch + " cus=" + std::to_string(prop.multiProcessorCount) + " format=3";
}

// The entries of a tuning cache: by log2 N and by the queue mode they were
// timed in (1: one shared queue; always 0 up to 2^14 items, where there is no
// choice).
typedef std::map<std::pair<int, int>, SizePlan> CacheLines;
std::pair<int, int> cache_entry(int k, bool shared) { return {k, k > paco::kChipMaxLog2 && shared ? 1 : 0}; }

// Tuning cache: a "key <device key>" line, then lines "log2N l1 l2 t shared";
// '#' starts a comment.  A file with another key (or none) is ignored, and
// rewritten after tuning.
void read_cache(const char *path, const std::string &key, CacheLines &plans)
{
    std::ifstream f(path);
    std::string line;
    bool keyed = false;
    while (std::getline(f, line)) {
        if (line.empty() || line[0] == '#') continue;
        if (line.compare(0, 4, "key ") == 0) {
            keyed = line.substr(4) == key;
            continue;
        }
        if (!keyed) continue;
        std::istringstream is(line);
        int k, shared;
        SizePlan sp;
        if (is >> k >> sp.l1 >> sp.l2 >> sp.t >> shared)
            if (k >= paco::kBatchMinLog2 && k <= paco::kBatchMaxLog2 && valid_plan(k, sp) &&
                (shared == 0 || shared == 1))
                plans[cache_entry(k, shared == 1)] = sp;
    }
}

bool write_cache(const char *path, const std::string &key, const CacheLines &plans)
{
    std::ofstream f(path);
    if (!f) return false;
    f << "# paco batched plan cache: log2N l1 l2 t shared (N1 = 2^l1, N2 = 2^l2, b = 2^t; shared: one work queue)\n";
    f << "key " << key << '\n';
    for (auto &kv : plans)
        f << kv.first.first << ' ' << kv.second.l1 << ' ' << kv.second.l2 << ' ' << kv.second.t << ' '
          << kv.first.second << '\n';
    return bool(f);
}

bool bad_ptr16(const void *p) { return !p || (reinterpret_cast<uintptr_t>(p) & 15); }

}  // namespace

extern "C" {

paco_status paco_batch_plan_create(paco_batch_plan **bp, int32_t count, const int64_t *N, paco_dtype dt,
                                   const char *tune_cache_path)
{
    return paco_batch_plan_create_ex(bp, count, N, dt, tune_cache_path, nullptr);
}

paco_status paco_batch_plan_create_ex(paco_batch_plan **bp, int32_t count, const int64_t *N, paco_dtype dt,
                                      const char *tune_cache_path, const paco_batch_options *options)
{
    if (!bp) return bfail(PACO_ERR_INVALID_ARG, "plan out-pointer is NULL");
    *bp = nullptr;
    const paco_batch_options opt = options ? *options : paco_batch_options{};
    if (opt.flags & ~(PACO_BATCH_NO_TUNE | PACO_BATCH_ONE_QUEUE | PACO_BATCH_SET_GAP))
        return bfail(PACO_ERR_INVALID_ARG, "unknown batch option flag");
    if ((opt.flags & PACO_BATCH_SET_GAP) && opt.gap < 0) return bfail(PACO_ERR_INVALID_ARG, "gap must be >= 0");
    if (opt.spin_limit >= (1u << 31)) return bfail(PACO_ERR_INVALID_ARG, "spin_limit must be below 2^31");
    if (dt == PACO_C64_MFMA_FP16X3 || dt == PACO_C64_MFMA_BF16X3 || dt == PACO_C64_MFMA_BF16X6)
        return bfail(PACO_ERR_UNSUPPORTED, "the batched form runs the FP32 arithmetic only");
    if (dt != PACO_C64) return bfail(PACO_ERR_INVALID_ARG, "unknown dtype");
    if (count < 1 || !N) return bfail(PACO_ERR_INVALID_ARG, "need count >= 1 and a size array");
    paco_batch_plan_s *P = new (std::nothrow) paco_batch_plan_s();
    if (!P) return bfail(PACO_ERR_ALLOC, "host allocation failed");
    P->count = count;
    P->opt = opt;
    std::vector<int> ks;
    for (int32_t i = 0; i < count; ++i) {
        const int k = paco::ilog2_pow2(N[i]);
        if (k < 0) {
            free_plan(P);
            return bfail(PACO_ERR_NOT_POWER_OF_B, "every size must be a power of two");
        }
        if (k < paco::kBatchMinLog2 || k > paco::kBatchMaxLog2) {
            free_plan(P);
            return bfail(PACO_ERR_UNSUPPORTED, "batched sizes must lie in [2^2, 2^20]");
        }
        P->N.push_back(N[i]);
        P->offset.push_back(P->total);
        P->total += N[i];
        if (std::find(ks.begin(), ks.end(), k) == ks.end()) ks.push_back(k);
    }
    std::sort(ks.begin(), ks.end());
    hipError_t e = hipGetDevice(&P->device);
    if (e != hipSuccess) {
        free_plan(P);
        return bhip(e, "hipGetDevice");
    }
    // per-size plans: cache file (lines of this batch's queue mode), then tuning
    // (unless PACO_BATCH_NO_TUNE), else defaults
    const Queues qorder = deal_queues(P);
    CacheLines lines;
    const std::string key = cache_key();
    if (tune_cache_path) read_cache(tune_cache_path, key, lines);
    std::vector<int> missing;
    for (int k : ks) {
        const auto at = lines.find(cache_entry(k, P->coh));
        if (at == lines.end()) missing.push_back(k);
        else P->plans[k] = at->second;
    }
    if (!missing.empty() && !(opt.flags & PACO_BATCH_NO_TUNE)) {
        paco_status st = tune(P, P->plans, missing);
        if (st != PACO_OK) {
            free_plan(P);
            return st;
        }
        for (int k : missing) lines[cache_entry(k, P->coh)] = P->plans[k];
        if (tune_cache_path && !write_cache(tune_cache_path, key, lines)) {
            free_plan(P);
            return bfail(PACO_ERR_INVALID_ARG, std::string("cannot write the tuning cache ") + tune_cache_path);
        }
    } else {
        for (int k : missing) P->plans[k] = paco::candidates(k).front();
    }
    paco_status st = build_batch(P, qorder);
    if (st != PACO_OK) {
        free_plan(P);
        return st;
    }
    paco::set_last_error("");
    *bp = P;
    return PACO_OK;
}

paco_status paco_batch_workspace_size(const paco_batch_plan *bp, size_t *bytes)
{
    if (!bytes) return bfail(PACO_ERR_INVALID_ARG, "bytes out-pointer is NULL");
    *bytes = 0;
    if (!bp) return bfail(PACO_ERR_INVALID_ARG, "plan is NULL");
    *bytes = size_t(bp->total) * 8;
    return PACO_OK;
}

paco_status paco_execute_batched(const paco_batch_plan *bp, const void *in, void *out, void *workspace,
                                 size_t workspace_bytes, void *stream)
{
    if (!bp) return bfail(PACO_ERR_INVALID_ARG, "plan is NULL");
    if (bad_ptr16(in) || bad_ptr16(out) || bad_ptr16(workspace))
        return bfail(PACO_ERR_INVALID_ARG, "in/out/workspace must be non-NULL and 16-byte aligned");
    const size_t need = size_t(bp->total) * 8;
    if (workspace_bytes < need) return bfail(PACO_ERR_WORKSPACE, "workspace smaller than the total items * 8 bytes");
    const uintptr_t wb = reinterpret_cast<uintptr_t>(workspace), ib = reinterpret_cast<uintptr_t>(in),
                    ob = reinterpret_cast<uintptr_t>(out);
    if ((wb < ib + need && ib < wb + need) || (wb < ob + need && ob < wb + need))
        return bfail(PACO_ERR_INVALID_ARG, "workspace overlaps in or out");
    if (ib != ob && ib < ob + need && ob < ib + need) return bfail(PACO_ERR_INVALID_ARG, "in and out overlap partially");
    hipError_t e = launch_batch(bp, in, out, workspace, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return bhip(e, "batched launch");
    return PACO_OK;
}

paco_status paco_batch_plan_describe(const paco_batch_plan *bp, int32_t index, int64_t *N1, int64_t *N2, int64_t *p,
                                     int32_t *b, char *buf, size_t buflen)
{
    if (!bp) return bfail(PACO_ERR_INVALID_ARG, "plan is NULL");
    if (index >= bp->count) return bfail(PACO_ERR_INVALID_ARG, "index out of range");
    if (index >= 0) {
        const int k = paco::ilog2_pow2(bp->N[index]);
        const SizePlan &sp = bp->plans.at(k);
        const int64_t n1 = int64_t(1) << sp.l1, n2 = int64_t(1) << sp.l2;
        if (N1) *N1 = n1;
        if (N2) *N2 = n2;
        // p has no effect on one device (the output is the same for every
        // valid p); the plan reports the largest p with slabs of at least 16
        // items (one 128-byte line), and at least 2
        if (p) *p = std::max<int64_t>(2, std::min(n1, n2) / 16);
        if (b) *b = 1 << sp.t;
    }
    if (buf && buflen) {
        std::strncpy(buf, bp->desc.c_str(), buflen - 1);
        buf[buflen - 1] = 0;
    }
    return PACO_OK;
}

paco_status paco_batch_errors(const paco_batch_plan *bp, uint32_t *count)
{
    if (!bp || !count) return bfail(PACO_ERR_INVALID_ARG, "plan or count is NULL");
    *count = 0;
    hipError_t e = hipMemcpy(count, bp->args.errors, sizeof(uint32_t), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return bhip(e, "hipMemcpy");
    return PACO_OK;
}

paco_status paco_batch_plan_destroy(paco_batch_plan *bp)
{
    free_plan(bp);
    return PACO_OK;
}

}  // extern "C"
