// Host side of the C ABI declared in include/gcoo.h: argument checks, device-buffer layout,
// kernel selection and launches.  No compute happens on the host.
#include "gcoo.h"

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>

#include <algorithm>
#include <array>
#include <atomic>
#include <chrono>
#include <cmath>
#include <memory>
#include <mutex>
#include <thread>
#include <type_traits>

#include "gcoo_band.hpp"
#include "gcoo_band_build.hpp"
#include "gcoo_build_kernels.hpp"
#include "gcoo_order_kernels.hpp"
#include "gcoo_sched.hpp"
#include "gcoo_sched_build.hpp"
#include "gcoo_share.hpp"
#include "gcoo_share_build.hpp"
#include "gcoo_spdm_launch.hpp"
#include "gcoo_spdm_lds_kernel.hpp"

namespace {

thread_local std::string g_hip_error;

int hip_fail(hipError_t e, const char* what)
{
    g_hip_error = std::string(what) + ": " + hipGetErrorString(e);
    return GCOO_EHIP;
}

#define HIP_TRY(expr)                                  \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return hip_fail(e_, #expr); \
    } while (0)

// A call that cannot be recorded into a graph says so before it launches anything: the replay of a kernel that reads or writes pinned
// memory of the library would meet what later calls have put there.
int refuse_capture(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(s, &status));
    return status == hipStreamCaptureStatusNone ? GCOO_OK : hip_fail(hipErrorStreamCaptureUnsupported, "call on a stream that is being captured");
}

constexpr size_t kAlign = 256;
size_t al(size_t bytes) { return (bytes + kAlign - 1) / kAlign * kAlign; }

constexpr int kMaxDevices = 64;

// A number that a kernel hands to the host in the middle of a call: the kernel writes it to pinned host memory, so that no copy
// stands between the kernel and the host's wait for the stream.  A call that goes on behind the kernel on its stream looks for the number there, for
// kHostLook, before it waits: the wait comes back 6 us after the number, since it takes the end of the kernel and the runtime's way from its signal
// (1777 x 2301, 3 %, N = 1117, conversion that reads the count and product: 53.0 and 47.7 us; count, conversion and product of a dense 4000 x 4000
// with 2 %: 161 and 154 us).  Such calls in a row find the product of the one before under way, hence as long a look as the shorter products take (100 us: 161).
// With the number there the work before the kernel has ended, and so have the kernel's reads.  kHostSlots such calls may be under way at once, over all devices and threads; a call takes a
// slot for its own use and gives it back when it returns, and waits for one while all are taken (fails where all are lost).  Each slot has words of device memory as
// well (per device, zero between calls), in which the workgroups of a kernel count themselves.  The pinned page is allocated once per process.
constexpr int kHostSlots = 64;
constexpr size_t kHostSlotWords = 8;
constexpr unsigned long long kHostNothing = ~0ull;
constexpr std::chrono::microseconds kHostLook(1000);
__device__ __align__(128) unsigned long long g_tickets[kHostSlots][(gcoo::kTicketWords + 1) * gcoo::kTicketStride];
std::atomic<uint64_t> g_slots_taken{0};
std::atomic<int> g_slots_lost{0};

class HostSlot {
public:
    ~HostSlot()
    {
        if (i_ >= 0) g_slots_taken.fetch_and(~(1ull << i_), std::memory_order_acq_rel);
    }
    // For a kernel on stream `s`.
    int claim(hipStream_t s)
    {
        const int rc = refuse_capture(s);
        if (rc != GCOO_OK) return rc;
        static std::mutex mutex;
        static unsigned long long* pinned = nullptr;
        static unsigned long long* tickets[kMaxDevices] = {};
        int dev = -1;
        HIP_TRY(hipGetDevice(&dev));
        if (dev < 0 || dev >= kMaxDevices) return GCOO_EINVAL;
        {
            std::lock_guard<std::mutex> lock(mutex);
            if (!pinned) {
                void* ptr = nullptr;
                HIP_TRY(hipHostMalloc(&ptr, kHostSlots * kHostSlotWords * 8, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent));
                pinned = static_cast<unsigned long long*>(ptr);
            }
            if (!tickets[dev]) {
                void* ptr = nullptr;
                HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_tickets)));
                tickets[dev] = static_cast<unsigned long long*>(ptr);
            }
            host_ = pinned;
            ticket_ = tickets[dev];
        }
        uint64_t taken = g_slots_taken.load(std::memory_order_relaxed);
        while (true) {
            if (taken == ~0ull) {
                if (g_slots_lost.load(std::memory_order_relaxed) == kHostSlots) return hip_fail(hipErrorUnknown, "all places for a number from the device are lost");
                std::this_thread::yield();
                taken = g_slots_taken.load(std::memory_order_relaxed);
                continue;
            }
            const int i = __builtin_ctzll(~taken);
            if (g_slots_taken.compare_exchange_weak(taken, taken | 1ull << i, std::memory_order_acq_rel)) { i_ = i; break; }
        }
        host_ += (size_t)i_ * kHostSlotWords;
        ticket_ += (size_t)i_ * (gcoo::kTicketWords + 1) * gcoo::kTicketStride;
        __atomic_store_n(host_, kHostNothing, __ATOMIC_RELEASE);
        return GCOO_OK;
    }
    unsigned long long* host() const { return host_; }
    gcoo::DenseTicket ticket() const { return {ticket_, gcoo::kTicketWords}; }
    // After the launch, in a call that goes on behind the kernel on its stream: looks for the number first.
    int look(hipStream_t s, unsigned long long* answer)
    {
        const auto until = std::chrono::steady_clock::now() + kHostLook;
        do {
            for (int i = 0; i < 64; ++i) {
                *answer = __atomic_load_n(host_, __ATOMIC_ACQUIRE);
                if (*answer != kHostNothing) return GCOO_OK;
                __builtin_ia32_pause();
            }
        } while (std::chrono::steady_clock::now() < until);
        return wait(s, answer);
    }
    // After the launch.  Where the wait fails nobody gets the slot again: the kernel may still write there.
    int wait(hipStream_t s, unsigned long long* answer)
    {
        const hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            lose();
            return hip_fail(e, "wait for a number from the device");
        }
        *answer = __atomic_load_n(host_, __ATOMIC_ACQUIRE);
        return GCOO_OK;
    }
    // An error behind the launch may be one of an earlier call of this thread, and the kernel on its way: the slot is given back when it has ended.
    void abandon(hipStream_t s)
    {
        if (hipStreamSynchronize(s) != hipSuccess) lose();
    }

private:
    void lose()
    {
        i_ = -1;
        g_slots_lost.fetch_add(1, std::memory_order_relaxed);
    }
    int i_ = -1;
    unsigned long long* host_ = nullptr;
    unsigned long long* ticket_ = nullptr;
};

// Pinned memory in which a host CSR input waits for the device: the call copies the caller's arrays there (5 us for half a
// megabyte, where a copy from pageable memory takes 17 to 25 us for each array) and need not wait for the device, whose kernels read them where
// they are or from one copy.  kStageSlots buffers of kStageBytes each, allocated when first needed and held until the process ends; a buffer is free
// again when the event behind its last reader has come.  Larger inputs, and calls that find all buffers in the hands of other threads, are
// copied from the caller's arrays.
constexpr int kStageSlots = 4;
constexpr size_t kStageBytes = 4u << 20;
class HostStage {
public:
    ~HostStage()
    {
        if (!slot_) return;
        // A call that failed: its launches may still read the buffer.  Where even the wait for them fails nobody gets the buffer again.
        if (hipDeviceSynchronize() == hipSuccess) give_back(false);
        (void)hipGetLastError();
    }
    // false: none to be had (or HIP failed, which the copies that follow will say)
    bool claim()
    {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess) return false;
        std::unique_lock<std::mutex> lock(mutex());
        Slot* found = nullptr;
        Slot* oldest = nullptr;
        for (Slot& s : slots()) {
            if (s.held) continue;
            if (!s.in_flight || hipEventQuery(s.event) == hipSuccess) { found = &s; break; }
            if (!oldest || s.turn < oldest->turn) oldest = &s;
        }
        (void)hipGetLastError();                              // (an event that has not come is no error)
        if (!found && !oldest) return false;
        slot_ = found ? found : oldest;
        slot_->held = true;
        if (!found) {
            lock.unlock();
            const hipError_t e = hipEventSynchronize(slot_->event);
            lock.lock();
            if (e != hipSuccess) { slot_->held = false; slot_ = nullptr; return false; }
        }
        slot_->in_flight = false;
        if (slot_->event && slot_->device != dev) { (void)hipEventDestroy(slot_->event); slot_->event = nullptr; }
        if (!slot_->event) {
            if (hipEventCreateWithFlags(&slot_->event, hipEventDisableTiming) != hipSuccess) slot_->event = nullptr;
            slot_->device = dev;
        }
        // (coherent whatever the process has as its default: kernels read what the host has written there since the last one did)
        if (!slot_->ptr && hipHostMalloc(&slot_->ptr, kStageBytes, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) slot_->ptr = nullptr;
        if (slot_->event && slot_->ptr) return true;
        (void)hipGetLastError();
        slot_->held = false;
        slot_ = nullptr;
        return false;
    }
    char* ptr() const { return static_cast<char*>(slot_->ptr); }
    explicit operator bool() const { return slot_ != nullptr; }
    // Behind the last launch that reads the buffer.  Without the event the buffer is kept, for the destructor to wait.
    hipError_t release(hipStream_t s)
    {
        const hipError_t e = hipEventRecord(slot_->event, s);
        if (e == hipSuccess) give_back(true);
        return e;
    }

private:
    struct Slot {
        void* ptr = nullptr;
        hipEvent_t event = nullptr;
        int device = -1;
        bool held = false, in_flight = false;
        uint64_t turn = 0;
    };
    static std::mutex& mutex() { static std::mutex m; return m; }
    static std::array<Slot, kStageSlots>& slots() { static std::array<Slot, kStageSlots> s; return s; }
    void give_back(bool in_flight)
    {
        static uint64_t turns = 0;
        std::lock_guard<std::mutex> lock(mutex());
        slot_->held = false;
        slot_->in_flight = in_flight;
        slot_->turn = ++turns;
        slot_ = nullptr;
    }
    Slot* slot_ = nullptr;
};

// Offsets of rows that do not descend and columns inside [0, k), without a branch per element.
bool csr_in_bounds(const int32_t* row_ptr, int64_t m, const int32_t* col_idx, int64_t nnz, int64_t k)
{
    int bad = 0;
    for (int64_t i = 0; i < m; ++i) bad |= row_ptr[i + 1] < row_ptr[i];
    if (bad) return false;
    const int32_t most = (int32_t)(k - 1);
    for (int64_t e0 = 0; e0 < nnz; e0 += 4096) {
        const int64_t e1 = e0 + 4096 < nnz ? e0 + 4096 : nnz;
        for (int64_t e = e0; e < e1; ++e) bad |= (col_idx[e] < 0) | (col_idx[e] > most);
        if (bad) return false;
    }
    return true;
}

// Scratch of gcoo_from_csr_device_static(), the conversion for callers that may not allocate device
// memory: the second buffer of the per-group radix sort (3 arrays of nnz words), which also holds the column bitmaps of the band
// schedule, and the counter from which the lists of a schedule take their place.  One copy per device, held until the process
// ends.  Host code never uses the array's name as an address: static_scratch() asks the runtime for
// the address on the current device, once per device, and everything goes through that pointer.
constexpr int64_t kStaticMaxNnz = 2 * 1024 * 1024;
constexpr size_t kStaticSortBytes = (size_t)kStaticMaxNnz * 4;        // each of the three arrays, a multiple of 256
constexpr size_t kStaticScratchBytes = 3 * kStaticSortBytes + 256;
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
std::mutex g_static_mutex;
unsigned char* g_static_ptr[kMaxDevices] = {};

int static_scratch(unsigned char** out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return GCOO_EINVAL;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        unsigned char* ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(g_static_scratch)));
        if (!ptr) return GCOO_EHIP;
        g_static_ptr[dev] = ptr;
    }
    *out = g_static_ptr[dev];
    return GCOO_OK;
}

// How the band schedule cuts a matrix: rows per wave and columns per lane (BandCut); h = 0: none is built.
struct BandPlan { int32_t h, v; };

// Carve-up of the caller's device buffer.  Offsets depend on (m, nnz, g) only.
struct Layout {
    size_t values, rows, cols, gIdxes, nnzPerGroup;        // the five arrays of the format
    size_t row_start, row_cols, row_vals, row_long;        // the entries in row order, the long rows (p <= 64; taller groups: in the inner handle)
    size_t sched_hdr, sched;                               // run schedule of the register kernel
    size_t order;                                          // groups by falling size, then those sizes (matrices of few groups)
    size_t share_ucols, share_ucount, share_hdr, share_blocks, share_sbase, share_alloc;   // share schedule (may be empty)
    BandPlan band;                                         // the band schedule
    size_t band_head, band_units, band_first, band_count;  // band schedule
    bool by_masks;                                         // a CSR input is ordered by take_rows and order_groups, else sorted by digits
    gcoo::OrderPlan plan;
    int64_t lists;                                         // workgroups of take_rows
    size_t take_flags, splits;
    size_t tmp_cols, tmp_rows, tmp_vals;                   // conversion scratch (second sort buffer)
    size_t in_row_ptr, in_cols, in_vals;                   // staging of a host CSR input
    size_t counter;                                        // device words: nnz (8 bytes), largest group (8), column-out-of-range flag (4), long rows (4), uneven rows (4), longest rows (4), ticket of a dense count (8)
    size_t persistent;                                     // bytes up to here stay in use after the conversion
    // offsets from here on are relative to the scratch area: the caller's buffer from `persistent` on, or the
    // library's static scratch
    size_t blk;                                            // dense input: entries per (group, column block)
    size_t total;
};

constexpr size_t kTicketAt = 32, kZeroedAt = 16;           // among the words of `counter`

// Column windows of the run schedule: bands of kWindowCols columns (a band of B of that many
// rows by one column tile stays in the L2 of the XCD working on the tile), at most kMaxWindows,
// and fewer when the matrix has so many groups that the per-window headers would dominate.
constexpr int64_t kWindowCols = 2048;

void pick_windows(int64_t k, int64_t g, int32_t* nw, int32_t* window_cols)
{
    const int64_t wc = kWindowCols;
    int64_t n = (k + wc - 1) / wc;
    const int64_t cap_groups = g > 0 ? (int64_t(1) << 22) / g : gcoo::kMaxWindows;
    int64_t cap = gcoo::kMaxWindows;
    if (cap_groups < cap) cap = cap_groups;
    if (cap < 1) cap = 1;
    if (n > cap) n = cap;
    if (n < 1) n = 1;
    *nw = (int32_t)n;
    *window_cols = (int32_t)((k + n - 1) / n > 0 ? (k + n - 1) / n : 1);
}

// Column blocks of the dense-input kernels: kDenseThreads*vw columns each.  The block table in the
// layout is sized for vw = 1 (the most blocks).
int64_t dense_blocks(int64_t k, int vw = 1) { return (k + gcoo::kDenseThreads * vw - 1) / (gcoo::kDenseThreads * vw); }

// 4 when rows of A can be read with 16-byte loads, else 1.
int dense_vec_width(const float* A, int64_t lda, int64_t k)
{
    return (k % 4 == 0 && lda % 4 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0) ? 4 : 1;
}

// Which schedules a conversion builds.  The automatic product runs the sixteen-wave kernel on the band schedule or works row by row,
// whichever band_time() and rows_time() below expect to be the faster; under GCOO_SHARE_AUTO a conversion builds the band schedule at most
// (and see share_schedule_wanted()).  The run schedule and the share schedule, and with them the register kernel and the workgroup-shared one, are reached
// through gcoo_set_share_policy() only.
std::atomic<int> g_share_policy{GCOO_SHARE_AUTO};
// A conversion lays its buffer out more than once (size check, handle, inner handle): it reads the policy once, when
// it starts, and every layout of that call uses that value, whatever another thread sets meanwhile.
thread_local int t_policy_of_call = -1;
struct PolicyOfCall {
    bool outermost;
    PolicyOfCall() : outermost(t_policy_of_call < 0) { if (outermost) t_policy_of_call = g_share_policy.load(std::memory_order_relaxed); }
    ~PolicyOfCall() { if (outermost) t_policy_of_call = -1; }
};
int share_policy_now() { return t_policy_of_call >= 0 ? t_policy_of_call : g_share_policy.load(std::memory_order_relaxed); }

bool share_schedule_possible(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    return p <= gcoo::kShareMaxP && k <= gcoo::kShareMaxK && nnz > 0 && m > 0 && k > 0;
}

// The shapes for which GCOO_VARIANT_SHARE can be asked for under the automatic policy, and for which gcoo_default_p() returns a height for the
// workgroup-shared kernel; density and shape only.  The lines lie where the workgroup-shared kernel overtook the register kernel; they are kept as a promise to
// callers, the automatic product does not go by them.
bool share_shape_preferred(int64_t m, int64_t k, int64_t nnz)
{
    if (m <= 0 || k <= 0 || nnz <= 0 || k > gcoo::kShareMaxK) return false;
    const double density = (double)nnz / ((double)m * (double)k);
    if (density > 0.06) return false;
    // Whole steps (conversion + product) of those two kernels on uniform random square matrices, n = 2000 .. 14000: the wider A, the
    // less of a column tile of B stays in an XCD's L2 between the groups that read it, and the sooner fetching each
    // row once per 8 groups pays for a second schedule (n = 8000, 0.5 %: 0.43 against 0.49 ms; n = 10000, 0.5 %: 1.0 against 1.23).
    if (k >= 7000) return density >= 0.0035;
    if (k >= 5500) return density >= 0.008;
    return k >= 3500 && density >= 0.015;
}

bool share_kernel_preferred(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    return share_schedule_possible(m, k, nnz, p) && share_shape_preferred(m, k, nnz);
}

BandPlan band_plan(int64_t m, int64_t k, int64_t nnz, int32_t p);

// The share schedule itself is built on request, and for a matrix of the rule above whose bitmaps do not fit the scratch that band_plan()
// has for them: one of fewer than about 1 / (6 density) rows, 48 at 0.35 %.  No automatic product reads it there; GCOO_VARIANT_SHARE,
// which the rule promises, does.
bool share_schedule_wanted(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    const int policy = share_policy_now();
    if (policy == GCOO_SHARE_NEVER || !share_schedule_possible(m, k, nnz, p)) return false;
    return policy == GCOO_SHARE_ALWAYS || (share_kernel_preferred(m, k, nnz, p) && band_plan(m, k, nnz, p).h == 0);
}

// The run schedule is what GCOO_VARIANT_REG reads when the policy is not the automatic one.
bool run_schedule_wanted(int32_t p) { return p <= gcoo::kSchedMaxP && share_policy_now() != GCOO_SHARE_AUTO; }

// A workgroup of that kernel runs for a whole (super-group, column tile): how well `items` of them fill
// the 256 compute units, as the fraction of the rounds they need that is work.
double fill_of_rounds(int64_t items)
{
    if (items <= 0) return 0.0;
    const int64_t rounds = (items + 255) / 256;
    return (double)items / (double)(rounds * 256);
}

int64_t share_items(int64_t m, int32_t p, int64_t N)
{
    const int64_t g = (m + p - 1) / p;
    return gcoo::share_super_groups(g) * ((N + 255) / 256);
}

// Group height for the workgroup-shared kernel (the sixteen-wave kernel cuts the rows by itself, band_plan()): taller groups mean fewer rows of B fetched per
// multiply-add, but the workgroups must fill their rounds over the compute units.  The time of a launch goes
// like rounds x (time of a workgroup), and the time of a workgroup like p plus a part that does not depend
// on p (the per-band steps); measured best heights: 42 at 8000 x 8000 (768 workgroups = 3 rounds), 48 at
// 14000 x 14000, 32 at 4000 x 4000 (256 workgroups), which this rule reproduces.
int32_t share_best_p(int64_t m, int64_t N)
{
    int32_t best = 32;
    int64_t best_cost = INT64_MAX;
    for (int32_t p = gcoo::kShareMaxP; p >= 24; --p) {
        const int64_t rounds = (share_items(m, p, N) + 255) / 256;
        const int64_t cost = rounds * (p + 24);
        if (cost < best_cost) { best_cost = cost; best = p; }
    }
    return best;
}

// Times of the two kernels that the automatic choice is between, in microseconds: fitted to 492 products by the row-by-row kernel and 906 by the two cuts of the bands, on uniform random
// matrices (1200 to 15000 rows and columns, 4 to 250 entries per row and up to 20 % dense, N = 300 to 15000, B not in a cache), half of them with rows of B on 128-byte lines (`lines`) and half
// inside; mean error 5 to 8 %.  The row-by-row kernel has had other tiles since (spdm_rows.hip): over 1237 drawn products of more than 1200 rows its time is 3 % short on average, mean error 13 %.  Choosing among the three
// kernels by these times took 0.6 % longer than always the fastest over 1600 drawn products, 1.0 % over the 579 of them with a band schedule.
// `outside`: how much of B is beyond what the memory-side cache holds of it beside C.
double outside_cache(int64_t k, int64_t N)
{
    const double big = ((double)k * (double)N - 4e7) / 6e7;
    return big < 0.0 ? 0.0 : (big > 1.0 ? 1.0 : big);
}
// Row by row: the bytes of B that the entries take through the vector caches, slower the less of a tile of B stays in an XCD's L2 and
// where rows of B begin inside a 128-byte line; C and B once.
double rows_time(int64_t m, int64_t k, int64_t nnz, int64_t N, bool lines)
{
    const double row = 4.0 * (double)N, md = (double)m, kd = (double)k, taken = (double)nnz;
    if (lines) return 2.5 + row * (taken * (1.0 + std::pow(kd / 49100.0, 0.974)) / 31.8e6 + md / 6.6e6 + kd / 5.2e6 + outside_cache(k, N) * (md + kd) / 31.8e6);
    return 2.4 + row * (taken * (1.0 + std::pow(kd / 13200.0, 1.49)) / 29.3e6 + md / 5.9e6 + kd / 4.9e6);
}
// The same for matrices of so few columns that the tile kernel is the other choice (k <= 2500 or so, cache-resident, fitted to 1336 products of 100 to 20000 rows, N = 16 to 8000, mean error 8 %):
// what its slots take of B is whole tiles, and launches of few workgroups leave compute units idle.  The widths here are those of the kernel that was fitted, not those that launch_spdm_rows() takes now, with which
// it needs 14 to 18 % less than this on average (mean error 15 to 18 %, 1700 drawn products).
double few_columns_rows_time(int64_t m, int64_t k, int64_t nnz, int64_t N, bool lines)
{
    const int64_t tile = N <= 16 ? 16 : (N <= 32 ? 32 : (N > 64 && k <= (lines ? 4096 : 6500) ? 128 : 64)), tiles = (N + (lines ? 0 : 31) + tile - 1) / tile;
    const double mean = (double)nnz / (double)m;
    return 4.2 + 4.0 * ((double)nnz * (double)(tiles * tile) / (lines ? 32.2e6 : 28.2e6) + (double)m * (double)N / 5.0e6) + 0.0044 * std::min(mean, 400.0);
}
// How the tile kernel cuts a product, and the time that this takes; row_wgs = 0: it does not serve the shape.  A round of the launch over the compute units, two workgroups to one
// where their LDS allows it, costs 1.5 us and what the tiles take to come in, and the entries of its rows: 3.8 ns per sixteen of them while enough waves read LDS, 26 ns per entry of a row for
// a wave by itself.  Where rows are long and workgroups have fewer of them than slots, a row has a whole wave to itself (`whole`; 1000 x 2480, 20 %, N = 64: 19.7 us with a row per slot, 9.1 so).
// Fitted to the products above in 2 to 14 cuts each: mean error 8 %; the cut so chosen takes 1.3 % longer than the best one.
// `preferred`: the tile kernel is taken, [1] where rows of B are on lines: where it is expected to need 0.85 of few_columns_rows_time(), which is about what the row-by-row kernel
// really takes: of 900 drawn products of up to 2558 columns 29 lose more than 3 % by the choice, 7 more than 10 %, and all take 0.5 % longer than by the faster of the two.
struct TilePlan { int64_t row_wgs; bool whole; double time; bool preferred[2]; };
const TilePlan& tile_plan(int64_t m, int64_t k, int64_t nnz, int64_t N)
{
    // (a product asks more than once, and a small one is not long)
    static thread_local struct { int64_t m, k, nnz, N; TilePlan plan; } last = {0, 0, 0, 0, {0, false, 0.0, {false, false}}};
    if (last.m == m && last.k == k && last.nnz == nnz && last.N == N) return last.plan;
    TilePlan best = {0, false, 0.0, {false, false}};
    if (m >= 1 && k >= 1 && N >= gcoo::kTileCols && nnz <= gcoo::kTileMaxNnz) {
        const int64_t tiles = (N + gcoo::kTileCols - 1) / gcoo::kTileCols, most_rows = gcoo::tile_most_rows(k), least = most_rows >= 1 ? (m + most_rows - 1) / most_rows : 0;
        const double mean = (double)nnz / (double)m;
        const int64_t wanted[] = {least, 256 / tiles, 512 / tiles, 768 / tiles, 1024 / tiles, m / 512, m / 256};
        for (int64_t wgs : wanted) {
            if (least < 1 || wgs < least) continue;
            const int64_t rows = (m + wgs - 1) / wgs, total = tiles * ((m + rows - 1) / rows);
            if (total > 0x7ffffff0LL) continue;
            const int64_t per = gcoo::tile_lds(k, rows) <= gcoo::kTileLdsBytes / 2 - 16 && total > 256 ? 2 : 1, rounds = (total + 256 * per - 1) / (256 * per);
            for (int whole = 0; whole <= (mean >= 24.0 ? 1 : 0); ++whole) {
                const double items = whole ? (double)rows : (double)((rows + gcoo::kTileCols - 1) / gcoo::kTileCols), steps = whole ? std::ceil(mean / 16.0) : mean;
                const double full = (double)per * items * (steps + (whole ? 12.0 : 0.0)) * 0.0038, alone = std::ceil(items / 16.0) * (steps * 0.026 + (whole ? 0.52 : 0.38));
                const double t = 2.4 + (double)rounds * (1.54 + 0.00098 * (double)(k * per) + std::max(full, alone)) + 1e-6 * (double)m * (double)N;
                if (best.row_wgs == 0 || t < best.time) best = {wgs, whole != 0, t, {false, false}};
            }
        }
    }
    if (best.row_wgs > 0)
        for (int lines : {0, 1}) best.preferred[lines] = best.time < 0.85 * few_columns_rows_time(m, k, nnz, N, lines != 0);
    last = {m, k, nnz, N, best};
    return last.plan;
}
// The faster of the two without a schedule.
double no_schedule_time(int64_t m, int64_t k, int64_t nnz, int64_t N, bool lines)
{
    const double rows = rows_time(m, k, nnz, N, lines);
    const TilePlan& plan = tile_plan(m, k, nnz, N);
    return plan.preferred[lines] ? std::min(rows, plan.time + 1.0) : rows;
}
// Bands: a workgroup per compute unit and round; 0.63 us for a band by itself (80 KB of B, the barrier, the bubble behind it) and 2.46 ns per
// entry of the block, 0.67 and 1.64 in the tall cut, whose bands have twice the rows and whose tiles are half as wide; C and B once, and
// more for both when they do not fit the memory-side cache.  The tall cut is bound by what it fetches, which the compute units share, rather than by its last round: that
// counts in full for one round and less the more there are.  With more than 40 entries per (wave, band) the multiply-adds, which a compute unit has to itself, come
// near that bound, and the last round counts for half of what was left out (10000 x 10000, 0.75 %, heights of 48, 44 and 40, that is 4.3, 4.6 and 4.9 rounds: 804 750 753 us;
// 9600 x 9600, 0.9 %, 44 and 48, 4.1 and 3.8 rounds: 798 683).
double band_time(int64_t m, int64_t k, int64_t nnz, int64_t N, BandPlan plan, bool lines)
{
    const int64_t blocks = gcoo::band_blocks(m, plan.h), tile = 64 * plan.v, tiles = (N + tile - 1) / tile, rounds = (blocks * tiles + 255) / 256;
    const double row = 4.0 * (double)N, md = (double)m, kd = (double)k, block_rows = (double)(gcoo::kBandWaves * plan.h), outside = outside_cache(k, N) * (md + kd);
    const double entries = plan.v == 4 || md < block_rows ? (double)nnz / (double)blocks : (double)nnz / md * block_rows;       // of a full block
    const double bands = std::ceil(kd * -std::expm1(-entries / kd) / gcoo::band_rows_of(plan.v));                  // distinct columns of a block
    if (plan.v == 4) {
        if (lines) return 3.6 + (double)rounds * (0.628 * bands + 0.00246 * entries) + row * (md / 8.8e6 + kd / 5.3e6 + outside / 9.7e6);
        return 2.9 + (double)rounds * (0.637 * bands + 0.00246 * entries) + row * (md / 3.7e6 + kd / 6.7e6 + outside / 12.8e6);
    }
    const double full = md / block_rows * (double)tiles / 256.0, part = rounds > 1 ? 1.2 / (double)rounds : 1.0;
    const double turns = full + ((double)rounds - full) * (gcoo::band_entries(m, k, nnz, plan.h, 2) > 40.0 ? 0.5 + 0.5 * part : part);
    if (lines) return 1.1 + turns * (0.676 * bands + 0.00166 * entries) + row * (md / 6.0e6 + kd / 6.7e6 + outside / 18.1e6);
    return 0.3 + turns * (0.657 * bands + 0.00161 * entries) + row * (md / 2.8e6 + kd / 8.1e6 + outside / 18.6e6);
}

// The band schedule of a matrix, if it gets one.  The width of B is not known here: the blocks are cut so that a
// product with N = k is fastest, and the schedule is built where that product gains more by it than a conversion
// pays for it (12 us), or where GCOO_VARIANT_SHARE has to be served.
// The tall cut fetches half as much and has half as many barriers, but reads LDS eight bytes at a time, which takes as long as sixteen.  It is
// taken where its expected time is not the longer one (by more than 2 %), and never above
// 66 entries per (wave, band) (product alone, us, wide and tall; 8000 x 8000, 0.35 %: 295 275, 0.5 %: 333 294, 0.9 %: 420 405, 1.2 %: 480 487; 12000 x 12000, 0.2 %: 809 669, 0.5 %: 1153 874, 0.9 %:
// 1417 1309; 4000 x 4000, 0.5 %: 59 51, 2 %: 103 109; 14000 x 14000, 0.75 %: 2088 1845; 0.3 %, N = 500: 92 64).  Over 199 matrices with N near k the cut so chosen takes 0 to 0.7 % longer than the
// faster of the two.
// Fewer than 12 rows per wave only as long as the blocks before did not fill the compute units once: a matrix of few rows has few blocks (us, the best of 12 rows and more, and so:
// 1836 x 2885, 20 %: 203 126; 558 x 4511, 6.6 %, N = 1504: 125 42; 2447 x 1964, 12 %: 92 71; 2467 x 3522, 3.6 %: 81 71; 765 x 6196, 9.4 %: 227 199).
BandPlan band_plan(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    if (p > gcoo::kSchedMaxP || m <= 0 || k <= 0 || nnz <= 0 || k > gcoo::kBandMaxK || share_policy_now() == GCOO_SHARE_NEVER) return {0, 0};
    const bool asked = share_kernel_preferred(m, k, nnz, p);
    const bool lines = k % 32 == 0;
    // (a conversion asks for every layout it makes: the last answer of this thread is kept)
    static thread_local struct { int64_t m, k, nnz; bool asked; BandPlan plan; } last = {0, 0, 0, false, {0, 0}};
    if (last.m == m && last.k == k && last.nnz == nnz && last.asked == asked) return last.plan;
    last = {m, k, nnz, asked, {0, 0}};
    if (!asked && (rows_time(m, k, nnz, k, lines) < 30.0 || no_schedule_time(m, k, nnz, k, lines) < 30.0)) return last.plan;
    BandPlan best = {0, 0};
    double best_time = 0.0;
    for (int v : {4, 2}) {
        if (v == 2 && (best.h == 0 || k > gcoo::kBandTallMaxK)) break;
        const int64_t tiles = (k + 64 * v - 1) / (64 * v);
        for (int32_t h = 96 / v; h >= 1; --h) {
            if (h < 12 && gcoo::band_blocks(m, h + 1) * tiles >= 256) break;
            // the columns of every list's rows as a bitmap, in the second sort buffer
            if (h % gcoo::band_lists_of(v) || gcoo::band_lists(m, h, v) * ((k + 31) / 32) > 3 * nnz) continue;
            const BandPlan plan = {h, v};
            const double entries = gcoo::band_entries(m, k, nnz, h, v);
            if (v == 2 && entries > 66.0) continue;
            const double t = band_time(m, k, nnz, k, plan, lines), least = best.v == v ? best_time : 1.02 * best_time;
            if (best.h == 0 || t < least) { best_time = t; best = plan; }
        }
    }
    if (best.h && !asked && best_time + 12.0 > no_schedule_time(m, k, nnz, k, lines)) best = {0, 0};
    last = {m, k, nnz, asked, best};
    return best;
}

// Distinct columns that band_fill holds at a time: all, or as many as fit `lds` bytes.
constexpr size_t kBandFillMaxLds = 150 * 1024;
int64_t band_fill_chunk(int64_t k, int v, size_t lds)
{
    const int64_t band_rows = gcoo::band_rows_of(v);
    int64_t chunk = gcoo::band_max_bands(k, v) * band_rows;
    if (chunk > gcoo::kBandChunk) chunk = gcoo::kBandChunk;
    while (chunk > 0 && gcoo::band_fill_lds(k, chunk, v) > lds) chunk -= band_rows;
    return chunk;
}

// Whether order_groups and band_fill are one launch, in 49 KB of LDS, which with 3 KB of their own variables leave a compute unit room for three workgroups (52 KB, room for two:
// 8000 x 8000, 0.5 %, p = 42: 28.7 us, 24.9 so; 7000 x 7000, 0.35 %: 24.0 20.2).  More columns than those hold at a time cost
// another turn through the entries: that is worth it up to about two such turns, three where a group has few entries, and only for lists of up to 4096
// entries, twice what the threads keep.  order_plan() makes one more exception, where the distinct columns have the masks and a group has more than 800 entries and up to
// twelve columns for each: there a part of twice the entries holds too much of the heaviest groups of power-law rows (exponent 1.5, at most 4096).  The host does not know
// whether rows are uneven, so uniform matrices of that shape stay outside as well, and power-law rows of another shape are inside.
// Conversion, us, as two launches and as one: 3000 x 3000, 3 %: 23.9 15.9; 5000 x 5000, 0.3 %: 24.0 14.9; 4000 x 4000, 5 %: 32.8 23.8; 8000 x 8000, 2 %: 43.8 38.7; 5 %: 81 76;
// 14000 x 14000, 0.2 %: 49 31; 2 %: 104 116.  With the distinct columns' masks and up to twelve columns per entry: power-law rows, 9000 x 9000: 26 29, 12000 x 10000: 30 32,
// 14000 x 14000: 37 40, but 16384 x 16384: 35 to 46 and 38 to 50; uniform, 8000 x 8000, 0.44 %: 30 23, 14000 x 14000, 0.3 %: 53 43, 20000 x 16000, 0.32 %: 78 68.
// Power-law rows of exponent 1.3, masks for all columns: 12000 x 10000 40 49, 9000 x 9000 36 41, 4000 x 4000 25 25.
constexpr size_t kBothMaxLds = 49 * 1024;
bool order_and_fill_wanted(int64_t m, int64_t k, int64_t nnz, int64_t mean, BandPlan band)
{
    const int64_t chunk = band_fill_chunk(k, band.v, kBothMaxLds);
    if (chunk >= k) return true;
    return nnz / (gcoo::band_blocks(m, band.h) * gcoo::kBandWaves) <= 4096 && (9 * chunk >= 4 * k || (3 * chunk >= k && k > 12 * mean));
}

// How a CSR input of this shape is put into the order of the groups; false: sorted by digits of the column.  A part has up to 4096
// columns of at most 32 rows (2048 of 64, 512 of 256: 16 KB of masks) and fewer where it would hold more than 1024 entries on
// average (4000 x 4000, 5 %, us for 2048, 1024, 512, 256: 11.4, 11.4, 14.2, 21.2; 1777 x 2301, 3 %: 13.8, 9.0, 8.2, 7.9).  The launch that fills the bands as well
// has 512 threads for a part, which holds twice as many (500 and 1000 parts there: 12.4 and 14.4 us with 512 threads, 11.7 with 256).
// With more than 5.5 columns per entry of a group the distinct columns have the masks, not all of them, unless the whole conversion is one launch:
// parts of up to 16384 columns, and fewer where a part would hold more than 640 entries, 400 up to twelve columns per entry: there one of a matrix with power-law
// rows holds many times the mean (640 and 400: 20000 x 16000, 0.1 % (31): 44 51; power-law rows, 11370 x 14582 (9): 39 35, 12000 x 10000 (6): 44 32)
// (in a launch of its own up to fourteen columns per entry: power-law rows of up to 20000 columns are there, and three parts are not enough for the heavy groups; 640 and 400:
// power-law rows, 20000 x 20000 (13.2): 61 42, 17000 x 20000 (12.9): 58 39; but 20000 x 20000, 0.24 % (13): 67 72, 16000 x 16000, 0.24 % (13): 48 54)
// (whole conversion, us, by masks or, beyond 32 columns per entry, by digits, and so; columns per entry in brackets: 12001 x 12001, 0.05 % (62): 21 12;
// 20000 x 20000, 0.05 % (62): 65 49; 8000 x 8000, 0.1 % (31): 14.3 12.2; 0.2 % (16): 29.6 27.6; 0.5 % (6): 33.3 33.3; power-law rows of exponent 1.5, 9000 x 8500 (5.3): 32.1 37.6,
// 7577 x 7577 (4.7): 33.7 39.0.  With the other steps since, two or three matrices each: 16384 x 16384 (10): 43 42, from 0.86x to 1.04x for one matrix; 20000 x 15000 (9): 50 49;
// 12000 x 10000 (8): 35 30; 9000 x 9000 (5.6): 33 26; 20000 x 20000 (13): 49 42.  Rows of exponent 1.6 and 1.8, whose heaviest groups are a large share of all entries, are
// slower so: 16384 x 16384 39 91 and 37 49, 9000 x 9000 31 39 and 24 42: one workgroup goes through such a group).
//
// Where a group's masks and entries fit the LDS of a workgroup and nothing else is to be made of the rows, one launch is the whole conversion (conversion and
// product, us, by take_rows and order_groups and so; 600 x 600, 5 %, N = 600: 17.7 12.4; 1000 x 1000, 5 %: 25.7 20.8; 2500 x 2500, 1 %, N = 1024: 26.9 21.7, from host
// memory 48.0 35.7; 1777 x 2301, 3 %, N = 1117: 40.9 36.4; 16000 x 300, 15 %, N = 64: 31.8 20.0; power-law rows, 2000 x 1300, N = 1000: 46.6 36.2).  It has 1024 threads for a
// large group, and for one of many columns while the groups are one to a compute unit (this launch, 256 and 1024 threads: 927 x 655, 16 %: 11.9 8.6; 2500 x 2500, 1 %: 8.6 7.9;
// 256 x 4000, 1 %: 9.1 8.0; but 1000 x 1000, 2 %: 6.4 7.2; 256 x 256, 10 %: 6.2 6.9; 9000 x 1000, 2 %, and product, N = 64: 12.9 15.8).
constexpr int64_t kOrderLds = 61 * 1024;                  // dynamic LDS of order_groups, at most
bool order_plan(int64_t m, int64_t k, int64_t nnz, int32_t p, BandPlan band, bool marked, gcoo::OrderPlan* plan)
{
    *plan = {};
    if (m <= 0 || k <= 0 || nnz <= 0) return false;
    const int64_t g = (m + p - 1) / p, mean = nnz / g + 1;
    if (k > 128 * mean) return false;
    const int32_t words = p <= 32 ? 1 : (p <= 64 ? 2 : 8), most = words == 1 ? 12 : (words == 2 ? 11 : 9);
    const bool ranked = 2 * k > 11 * mean && (k > ((int64_t)1 << most) || band.h > 0 || run_schedule_wanted(p));
    int32_t shift = ranked ? 5 : 0;
    while (((int64_t)1 << shift) < k && shift < (ranked ? 14 : most)) ++shift;
    // entries, of eight bytes, that the LDS holds beside the masks of a part's columns (the largest groups that go in one launch, us, in two and so: 3000 x 1000, 16 % (5180 per group): 14.8 9.9;
    // 3000 x 2500, 3 % (2440): 13.0 7.0; 1000 x 2000, 6 % (4020): 11.1 7.5)
    const auto room_at = [&](int32_t shift) { return (kOrderLds - 4 * (((int64_t)1 << shift) * (words + 1) + 2 * 1024)) / 8; };
    const int64_t room = room_at(shift);
    const bool fused = !ranked && k <= ((int64_t)1 << most) && mean + mean / 16 <= room && band.h == 0 && !run_schedule_wanted(p);
    const int32_t threads = fused && (mean > 2048 || (g <= 256 && ((int64_t)words << shift) >= 4096)) ? 1024 : gcoo::kOrderThreads;
    const bool both = marked && words <= 2 && !(ranked && k <= 12 * mean && mean > 800) && order_and_fill_wanted(m, k, nnz, mean, band);
    const int64_t each = !ranked ? 1024 : (k > (both ? 12 : 14) * mean ? 640 : 400);              // entries of a part
    while (!fused && shift > 7 && (mean << shift) / k > each * (both ? 2 : 1)) --shift;
    const int64_t parts = (k + ((int64_t)1 << shift) - 1) >> shift;
    if (parts > gcoo::kOrderMaxParts || parts * g > 0x7fffffffLL) return false;
    // lists of rows of take_rows: those of the band schedule, else enough workgroups for four per compute unit
    int64_t rows = (m + 1023) / 1024;
    rows = band.h > 0 ? band.h / gcoo::band_lists_of(band.v) : (rows > 64 ? 64 : rows);
    int64_t cap = mean / parts * 3 / 2 + 64;
    const int64_t most_cap = fused ? room : (both ? room_at(shift < most ? shift : most) : gcoo::kOrderMaxCap);
    cap = cap < 256 ? 256 : (cap > most_cap ? most_cap : cap);
    // Distinct columns of a window: uniform parts have a few hundred, and the fewer, the more workgroups fit a compute unit; heavy groups go through their entries once more for
    // every further window (us for 4096, 2048, 1024: 12000 x 12000, 0.3 %: 38.9 34.6 34.6; power-law rows, 16384 x 16384, six draws: 42.2 41.1 48.3).
    const int32_t keys = ranked ? (int32_t)1 << std::min({shift, most, 11}) : 0;
    *plan = {shift, (int32_t)parts, (int32_t)rows, (int32_t)((cap + 3) / 4 * 4), fused, keys, both ? gcoo::kBothThreads : threads, both};
    return true;
}

// (device offsets that contradict each other may make more rows long than these: the rest are not listed)
int32_t long_room(int64_t m, int64_t nnz) { return (int32_t)(nnz / gcoo::rows_long(m, nnz)) + 1; }

Layout make_layout(int64_t m, int64_t k, int64_t nnz, int64_t g, int32_t p, bool scratch_inside = true)
{
    int32_t nw, wc;
    pick_windows(k, g, &nw, &wc);
    Layout L{};
    size_t at = 0;
    auto take = [&](size_t bytes) { size_t o = at; at += al(bytes ? bytes : 1); return o; };
    const size_t n4 = (size_t)nnz * 4;
    // the arrays whose size does not depend on nnz come first, so that a dense input can be
    // counted into them before nnz is known
    L.gIdxes = take((size_t)(g + 1) * 4);
    L.nnzPerGroup = take((size_t)g * 4);
    L.counter = take(kZeroedAt + 4 * gcoo::kSoonWord + 4);
    L.blk = take((size_t)g * (size_t)dense_blocks(k) * 4);
    L.values = take(n4);
    L.rows = take(n4);
    L.cols = take(n4);
    const bool rows = p <= gcoo::kSchedMaxP;
    L.row_start = take((size_t)(m + 1) * 4);
    L.row_cols = take(rows ? n4 : 0);
    L.row_vals = take(rows ? n4 : 0);
    L.row_long = take(rows ? (size_t)long_room(m, nnz) * 4 : 0);
    const bool sched = run_schedule_wanted(p);
    L.sched_hdr = take(sched ? (size_t)g * nw * gcoo::kMaxRun * sizeof(gcoo::SchedClass) : 0);
    L.sched = take(sched ? (size_t)gcoo::sched_words(nnz, g, nw) * 4 : 0);
    L.order = take(sched && g <= gcoo::kOrderMaxGroups ? (size_t)g * 8 : 0);
    const bool share = share_schedule_wanted(m, k, nnz, p);
    const int64_t nQ = gcoo::share_super_groups(g);
    L.share_ucols = take(share ? n4 : 0);
    L.share_ucount = take(share ? (size_t)nQ * 4 : 0);
    L.share_hdr = take(share ? (size_t)gcoo::share_hdr_words(nnz, g) * 4 : 0);
    L.share_blocks = take(share ? (size_t)gcoo::share_stream_blocks(nnz, g, k) * gcoo::kShareBlockWords * 4 : 0);
    L.share_sbase = take(share ? (size_t)nQ * gcoo::kShareW * 4 : 0);
    L.band = band_plan(m, k, nnz, p);
    const int64_t lists = L.band.h ? gcoo::band_blocks(m, L.band.h) * gcoo::kBandWaves : 0;
    L.band_head = take(L.band.h ? (size_t)(lists * gcoo::band_head_stride(k, L.band.v)) * gcoo::kBandHeadWords * 4 : 0);
    L.band_units = take(L.band.h ? (size_t)gcoo::band_units(nnz, m, k, L.band.h, L.band.v) * gcoo::kBandUnitWords * 4 : 0);
    L.band_first = take((size_t)lists * 4);
    L.band_count = take((size_t)(lists / gcoo::kBandWaves) * 4);
    L.by_masks = order_plan(m, k, nnz, p, L.band, L.band.h > 0 && !share, &L.plan);
    L.lists = L.plan.fused ? g : lists ? gcoo::band_lists(m, L.band.h, L.band.v) : (L.by_masks ? (m + L.plan.list_rows - 1) / L.plan.list_rows : 0);     // (a band block has empty lists behind the last row)
    L.take_flags = take(L.by_masks ? (size_t)L.lists * 4 : 0);
    L.splits = take(L.by_masks ? (size_t)m * (size_t)(L.plan.parts - 1) * 4 : 0);
    L.persistent = at;
    if (!scratch_inside) {
        // the fixed carve-up of the static scratch (no staging of a host input there)
        L.tmp_cols = 0;
        L.tmp_rows = kStaticSortBytes;
        L.tmp_vals = 2 * kStaticSortBytes;
        L.share_alloc = 3 * kStaticSortBytes;
        L.in_row_ptr = L.in_cols = L.in_vals = 0;
        L.total = L.persistent;
        return L;
    }
    at = 0;
    L.share_alloc = take(4);
    L.tmp_cols = take(n4);
    L.tmp_rows = take(n4);
    L.tmp_vals = take(n4);
    L.in_row_ptr = take((size_t)(m + 1) * 4);
    L.in_cols = take(n4);
    L.in_vals = take(n4);
    L.total = L.persistent + at;
    return L;
}

// Groups taller than the fast kernels serve (p > 64) get a second, kernel-private copy of the matrix regrouped at
// kInnerP rows: the buffer of such a handle is its own layout followed by that of the inner handle.
constexpr int32_t kInnerP = 32;
bool wants_inner(int32_t p) { return p > gcoo::kSchedMaxP; }
size_t total_bytes(int64_t m, int64_t k, int64_t nnz, int32_t p, bool scratch_inside)
{
    const size_t own = make_layout(m, k, nnz, (m + p - 1) / p, p, scratch_inside).total;
    if (!wants_inner(p)) return own;
    return al(own) + make_layout(m, k, nnz, (m + kInnerP - 1) / kInnerP, kInnerP, scratch_inside).total;
}

bool dims_ok(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    return m >= 0 && k >= 0 && nnz >= 0 && p >= 1 && p <= GCOO_MAX_P && m <= INT32_MAX && k <= INT32_MAX &&
           nnz <= INT32_MAX;
}

int radix_passes(int64_t k)
{
    int bits = 0;
    while (bits < 31 && ((int64_t)1 << bits) < k) ++bits;   // column indices fit in `bits` bits
    int passes = (bits + 7) / 8;
    return passes < 1 ? 1 : passes;
}

}  // namespace

struct gcoo_matrix {
    // Everything below is set by the conversion and only read afterwards.
    int64_t m, k, nnz, g;
    int32_t p;
    int32_t nw, window_cols;
    bool has_sched;            // the run schedule of the register kernel was built
    bool has_share;            // the share schedule was built
    bool from_csr = false;     // the input was CSR (as opposed to dense)
    bool long_places = false;  // the long rows are in places of their groups, not counted (RowsArgs)
    bool share_preferred;      // GCOO_VARIANT_SHARE can be asked for and is what gcoo_spdm_pick() answers where B is wide enough
    int device;
    char* base;
    Layout L;
    // p > 64: the same matrix regrouped at kInnerP rows per group, with the schedules of the fast kernels, in the
    // part of the caller's buffer behind this handle's own; gcoo_spdm() multiplies with it.  Owned.
    gcoo_matrix* inner = nullptr;
    ~gcoo_matrix() { delete inner; }
    float* values() const { return reinterpret_cast<float*>(base + L.values); }
    int32_t* rows() const { return reinterpret_cast<int32_t*>(base + L.rows); }
    int32_t* cols() const { return reinterpret_cast<int32_t*>(base + L.cols); }
    int32_t* gIdxes() const { return reinterpret_cast<int32_t*>(base + L.gIdxes); }
    int32_t* nnzPerGroup() const { return reinterpret_cast<int32_t*>(base + L.nnzPerGroup); }
    gcoo::SchedClass* sched_hdr() const { return reinterpret_cast<gcoo::SchedClass*>(base + L.sched_hdr); }
    uint32_t* sched() const { return reinterpret_cast<uint32_t*>(base + L.sched); }
    int32_t* row_start() const { return reinterpret_cast<int32_t*>(base + L.row_start); }
    int32_t* row_cols() const { return reinterpret_cast<int32_t*>(base + L.row_cols); }
    float* row_vals() const { return reinterpret_cast<float*>(base + L.row_vals); }
    int32_t* long_rows() const { return reinterpret_cast<int32_t*>(base + L.row_long); }
    uint32_t* uneven() const { return reinterpret_cast<uint32_t*>(base + L.counter + 24); }
    uint32_t* soon() const { return bad_col() + gcoo::kSoonWord; }
    int32_t* long_count() const { return reinterpret_cast<int32_t*>(base + L.counter + 20); }
    uint32_t* band_head() const { return reinterpret_cast<uint32_t*>(base + L.band_head); }
    uint32_t* band_units() const { return reinterpret_cast<uint32_t*>(base + L.band_units); }
    int32_t* band_first() const { return reinterpret_cast<int32_t*>(base + L.band_first); }
    int32_t* band_count() const { return reinterpret_cast<int32_t*>(base + L.band_count); }
    bool has_rows() const { return p <= gcoo::kSchedMaxP; }
    bool has_order() const { return has_sched && g > 0 && g <= gcoo::kOrderMaxGroups; }
    int32_t* order() const { return reinterpret_cast<int32_t*>(base + L.order); }
    unsigned long long* stats() const { return reinterpret_cast<unsigned long long*>(base + L.counter); }
    uint32_t* take_flags() const { return reinterpret_cast<uint32_t*>(base + L.take_flags); }
    uint32_t* bad_col() const { return reinterpret_cast<uint32_t*>(base + L.counter + kZeroedAt); }
    int32_t* share_ucols() const { return reinterpret_cast<int32_t*>(base + L.share_ucols); }
    int32_t* share_ucount() const { return reinterpret_cast<int32_t*>(base + L.share_ucount); }
    uint32_t* share_hdr() const { return reinterpret_cast<uint32_t*>(base + L.share_hdr); }
    uint32_t* share_blocks() const { return reinterpret_cast<uint32_t*>(base + L.share_blocks); }
    int32_t* share_sbase() const { return reinterpret_cast<int32_t*>(base + L.share_sbase); }
    int64_t share_nq() const { return gcoo::share_super_groups(g); }
};

namespace {

gcoo::RowsOut rows_out(const gcoo_matrix* h)
{
    if (!h->has_rows()) return {};
    return {h->row_cols(), h->row_vals(), h->row_start(), h->long_rows(), h->long_count(), gcoo::rows_long(h->m, h->nnz), long_room(h->m, h->nnz)};
}

int new_handle(int64_t m, int64_t k, int64_t nnz, int32_t p, void* dev_buf, gcoo_matrix** out, bool scratch_inside = true)
{
    gcoo_matrix* h = new (std::nothrow) gcoo_matrix;
    if (!h) return GCOO_ENOMEM;
    h->m = m; h->k = k; h->nnz = nnz; h->p = p;
    h->g = (m + p - 1) / p;
    h->base = static_cast<char*>(dev_buf);
    h->L = make_layout(m, k, nnz, h->g, p, scratch_inside);
    h->has_share = share_schedule_wanted(m, k, nnz, p);
    h->share_preferred = (h->has_share || h->L.band.h > 0) && share_kernel_preferred(m, k, nnz, p);
    h->has_sched = run_schedule_wanted(p);
    pick_windows(k, h->g, &h->nw, &h->window_cols);
    if (hipGetDevice(&h->device) != hipSuccess) h->device = -1;
    *out = h;
    return GCOO_OK;
}

// share_fill may ask for more dynamic LDS than a kernel gets by default: raised once per device (a compute unit
// has 160 KB; the kernel's static variables take a little of it).
constexpr int kShareFillMaxLds = 156 * 1024;
hipError_t share_fill_lds_limit()
{
    static std::atomic<unsigned> done[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (done[dev].load(std::memory_order_acquire)) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gcoo::share_fill), hipFuncAttributeMaxDynamicSharedMemorySize, kShareFillMaxLds);
    if (e == hipSuccess) done[dev].store(1u, std::memory_order_release);
    return e;
}

hipError_t band_fill_lds_limit()
{
    static std::atomic<unsigned> done[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (done[dev].load(std::memory_order_acquire)) return hipSuccess;
    for (const void* f : {reinterpret_cast<const void*>(&gcoo::band_fill<4, 512, 8, false>), reinterpret_cast<const void*>(&gcoo::band_fill<4, 1024, 4, false>),
                          reinterpret_cast<const void*>(&gcoo::band_fill<2, 1024, 4, false>), reinterpret_cast<const void*>(&gcoo::band_fill<4, 512, 8, true>),
                          reinterpret_cast<const void*>(&gcoo::band_fill<4, 1024, 4, true>), reinterpret_cast<const void*>(&gcoo::band_fill<2, 1024, 4, true>)}) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBandFillMaxLds);
        if (e != hipSuccess) return e;
    }
    done[dev].store(1u, std::memory_order_release);
    return e;
}

gcoo::FillArgs fill_args(const gcoo_matrix* h, const char* scratch, bool both)
{
    const int v = h->L.band.v;
    gcoo::FillArgs f{};
    f.row_start = h->row_start(); f.row_cols = h->row_cols(); f.row_vals = h->row_vals(); f.m = h->m; f.k = h->k; f.h = h->L.band.h;
    f.chunk = (int32_t)band_fill_chunk(h->k, v, both ? kBothMaxLds : kBandFillMaxLds); f.parts = reinterpret_cast<const uint32_t*>(scratch + h->L.tmp_cols);
    f.head_stride = gcoo::band_head_stride(h->k, v); f.head = h->band_head(); f.units = h->band_units(); f.first = h->band_first(); f.count = h->band_count();
    if (both) { f.flags = h->take_flags(); f.flag_count = (int32_t)h->L.lists; f.heavy = gcoo::kHeavy; }
    else f.uneven = h->uneven();
    return f;
}

// The kernel-private schedules that a conversion ends with (see share_schedule_wanted(), run_schedule_wanted() and band_plan()), on the
// conversion's stream, so that the handle is never written again.
// `scratch`: the conversion's scratch area (the counter of share_fill sits in it).  `marked`: the bitmaps of the band schedule are there; `grouped`: those of fill_dense_groups().
int launch_build_schedule(const gcoo_matrix* h, char* scratch, hipStream_t s, bool marked = false, bool filled = false, bool grouped = false)
{
    uint32_t* share_alloc = reinterpret_cast<uint32_t*>(scratch + h->L.share_alloc);
    if (h->g > 0 && h->has_sched) {
        // the groups by falling size, where the matrix has few of them: a workgroup more of the small-workgroup
        // instance, a launch of its own beside the large-workgroup instance
        int32_t* order = h->has_order() ? h->order() : nullptr;
        if (h->nnz / (h->g * h->nw) <= 1024) {
            const dim3 grid((unsigned)(h->g * h->nw + (order ? (h->g + 255) / 256 : 0)));
            gcoo::build_schedule<256><<<grid, dim3(256), 0, s>>>(h->gIdxes(), h->rows(), h->cols(), h->values(), h->p, h->g, h->nw,
                                                                 h->window_cols, h->sched_hdr(), h->sched(), order, order ? order + h->g : nullptr);
        } else {
            const dim3 grid((unsigned)(h->g * h->nw));
            gcoo::build_schedule<1024><<<grid, dim3(1024), 0, s>>>(h->gIdxes(), h->rows(), h->cols(), h->values(), h->p, h->g, h->nw,
                                                                   h->window_cols, h->sched_hdr(), h->sched(), nullptr, nullptr);
            HIP_TRY(hipGetLastError());
            if (order) gcoo::group_order_by_size<<<dim3((unsigned)((h->g + 1023) / 1024)), dim3(1024), 0, s>>>(h->gIdxes(), (int32_t)h->g, order, order + h->g);
        }
        HIP_TRY(hipGetLastError());
    }
    if (h->g > 0 && h->has_share) {
        const size_t bitmap_bytes = (size_t)((h->k + 31) / 32) * 4;
        // the bitmaps of the groups, one workgroup each, where they fit the second sort buffer (free by now: 12 bytes
        // per entry); otherwise one workgroup per super-group marks all its entries itself
        uint32_t* parts = nullptr;
        if ((uint64_t)h->g * bitmap_bytes <= (uint64_t)h->nnz * 12u) {
            parts = reinterpret_cast<uint32_t*>(scratch + h->L.tmp_cols);
            gcoo::share_mark_groups<<<dim3((unsigned)h->g), dim3(gcoo::kShareBuildThreads), bitmap_bytes, s>>>(h->gIdxes(), h->cols(), h->k, parts);
            HIP_TRY(hipGetLastError());
        }
        gcoo::share_union<<<dim3((unsigned)h->share_nq()), dim3(gcoo::kShareBuildThreads), bitmap_bytes, s>>>(
            h->gIdxes(), h->cols(), h->g, h->k, gcoo::kShareW, h->share_ucols(), h->share_ucount(), share_alloc, parts);
        HIP_TRY(hipGetLastError());
        // LDS of share_fill: its per-band tables and room for the columns of a group of up to twice the mean size
        // (between 8 K and 28 K entries: two workgroups share a compute unit up to 80 KB each)
        const size_t table_bytes = 4 * (size_t)((h->k + gcoo::kShareBandRows - 1) / gcoo::kShareBandRows + 1) * 4;
        int64_t stage_cap = 2 * (h->nnz / h->g + 1);
        stage_cap = stage_cap < 8192 ? 8192 : (stage_cap > 28672 ? 28672 : stage_cap);
        if (table_bytes + (size_t)stage_cap * 4 > (size_t)kShareFillMaxLds) stage_cap = 0;
        const size_t fill_lds = table_bytes + (size_t)stage_cap * 4;
        HIP_TRY(share_fill_lds_limit());
        gcoo::share_fill<<<dim3((unsigned)(h->share_nq() * gcoo::kShareW)), dim3(gcoo::kShareBuildThreads), fill_lds, s>>>(
            h->gIdxes(), h->rows(), h->cols(), h->values(), h->p, h->g, h->k, h->share_ucols(), h->share_ucount(), h->share_hdr(),
            h->share_blocks(), h->share_sbase(), share_alloc, (int32_t)stage_cap);
        HIP_TRY(hipGetLastError());
    }
    if (h->L.band.h > 0 && !filled) {
        const int32_t rows = h->L.band.h;
        const int v = h->L.band.v;
        const unsigned lists = (unsigned)(gcoo::band_blocks(h->m, rows) * gcoo::kBandWaves), marks = (unsigned)gcoo::band_lists(h->m, rows, v);
        const size_t words = (size_t)((h->k + 31) / 32);
        uint32_t* parts = reinterpret_cast<uint32_t*>(scratch + h->L.tmp_cols);          // the second sort buffer, free by now
        if (!marked) gcoo::band_mark<<<dim3(marks), dim3(gcoo::kBandMarkThreads), words * 4, s>>>(h->row_start(), h->row_cols(), h->m, h->k, rows / gcoo::band_lists_of(v), parts,
                                                                                                                gcoo::band_heavy(h->nnz, marks), h->uneven());
        HIP_TRY(hipGetLastError());
        const bool large = v == 2 || h->nnz / lists > 4096;
        gcoo::FillArgs f = fill_args(h, scratch, false);
        if (grouped) { f.out = rows_out(h); f.g = h->g; f.p = h->p; f.says_uneven = h->uneven(); f.soon = h->soon(); f.flag_count = (int32_t)marks; f.heavy = (uint32_t)gcoo::band_heavy(h->nnz, marks); }
        HIP_TRY(band_fill_lds_limit());
        auto pick = [&](auto by_groups) {
            constexpr bool GROUPED = decltype(by_groups)::value;
            return v == 2 ? gcoo::band_fill<2, 1024, 4, GROUPED> : (large ? gcoo::band_fill<4, 1024, 4, GROUPED> : gcoo::band_fill<4, 512, 8, GROUPED>);
        };
        (grouped ? pick(std::true_type{}) : pick(std::false_type{}))
            <<<dim3(lists), dim3(large ? 1024 : 512), gcoo::band_fill_lds(h->k, f.chunk, v), s>>>(f);
        HIP_TRY(hipGetLastError());
    }
    return GCOO_OK;
}

}  // namespace

extern "C" {

int gcoo_set_share_policy(int policy)
{
    if (policy < GCOO_SHARE_AUTO || policy > GCOO_SHARE_NEVER) return GCOO_EINVAL;
    g_share_policy.store(policy, std::memory_order_relaxed);
    return GCOO_OK;
}

int32_t gcoo_default_p(int64_t m, int64_t k, int64_t nnz, int64_t N)
{
    if (m < 0 || k < 0 || nnz < 0 || N < 0) return 0;
    if (N > 0 && N % 4 == 0 && share_policy_now() != GCOO_SHARE_NEVER && share_shape_preferred(m, k, nnz)) {
        const int32_t p = share_best_p(m, N);
        const int64_t items = share_items(m, p, N);
        if (items >= 192 && (k >= 9000 || fill_of_rounds(items) >= 0.8)) return p;
    }
    // The tall accumulator file of the register kernel (it needs a run schedule; the automatic product does not depend on the height).  Between 6 % and
    // 12 % density most groups touch most columns, and what that kernel fetches falls with the number of groups: 38 rows beat 32 by
    // 8 .. 28 % from 6000 columns on (n = 6000 .. 14000, s = 0.9 and 0.93); at 20 % and more, and at n = 4000, the two are within a few
    // per cent either way.
    if (m > 0 && k >= 5000 && N % 4 == 0) {
        const double density = (double)nnz / ((double)m * (double)k);
        if (density > 0.06 && density <= 0.12) return 38;
    }
    return 32;
}

size_t gcoo_device_bytes(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    if (!dims_ok(m, k, nnz, p)) return 0;
    return total_bytes(m, k, nnz, p, true);
}

}  // extern "C"

namespace {

// gcoo_from_csr() and gcoo_from_csr_device().  nnz_known < 0: learn nnz from the input.
// static_scratch_ptr != nullptr: the conversion's scratch is that area instead of the tail of dev_buf (device input with
// nnz given only).
int from_csr(int64_t m, int64_t k, const int32_t* row_ptr, const int32_t* col_idx, const float* vals, int src_on_device,
             int64_t nnz_known, int32_t p, void* dev_buf, size_t dev_buf_bytes, void* stream, gcoo_matrix** out,
             unsigned char* static_scratch_ptr = nullptr)
{
    const PolicyOfCall policy_of_call;
    const bool inside = static_scratch_ptr == nullptr;
    if (!out) return GCOO_EINVAL;
    *out = nullptr;
    if (!row_ptr || !dev_buf || !dims_ok(m, k, 0, p)) return GCOO_EINVAL;
    if (reinterpret_cast<uintptr_t>(dev_buf) % kAlign) return GCOO_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);

    const int64_t g = (m + p - 1) / p;
    int64_t nnz;
    if (src_on_device && nnz_known >= 0) {          // everything the host can check, before the first launch
        if (nnz_known > 0 && (!col_idx || !vals)) return GCOO_EINVAL;
        if (dev_buf_bytes < total_bytes(m, k, nnz_known, p, inside)) return GCOO_ENOMEM;
    }
    // nnz and the size of the largest group are computed on the device and stay there (the counters
    // sit at an offset of the buffer that does not depend on nnz); the launches that need the
    // latter read it there.
    const Layout L0 = make_layout(m, k, 0, g, p, inside);
    if (dev_buf_bytes < L0.total) return GCOO_ENOMEM;
    unsigned long long* stats = reinterpret_cast<unsigned long long*>(static_cast<char*>(dev_buf) + L0.counter);
    if (src_on_device) {
        // With nnz given nothing is read back here; otherwise nnz comes back in one word.
        if (nnz_known >= 0) {
            nnz = nnz_known;
        } else {
            HostSlot slot;
            int rc = slot.claim(s);
            if (rc != GCOO_OK) return rc;
            gcoo::read_entry_count<<<dim3(1), dim3(1), 0, s>>>(row_ptr, m, slot.host());
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) { slot.abandon(s); return hip_fail(e, "read_entry_count"); }
            unsigned long long got = 0;
            rc = slot.look(s, &got);
            if (rc != GCOO_OK) return rc;
            if (got > (unsigned long long)INT32_MAX) return GCOO_EBOUNDS;
            nnz = (int64_t)got;
        }
    } else {
        if (row_ptr[0] != 0) return GCOO_EBOUNDS;
        if (!csr_in_bounds(row_ptr, m, nullptr, 0, k)) return GCOO_EBOUNDS;
        nnz = row_ptr[m];
        if (nnz > 0 && (!col_idx || !vals)) return GCOO_EINVAL;
        if (!csr_in_bounds(row_ptr, 0, col_idx, nnz, k)) return GCOO_EBOUNDS;
    }
    if (nnz > 0 && (!col_idx || !vals)) return GCOO_EINVAL;
    const Layout L = make_layout(m, k, nnz, g, p, inside);
    if (dev_buf_bytes < total_bytes(m, k, nnz, p, inside)) return GCOO_ENOMEM;
    int rc = src_on_device ? GCOO_OK : refuse_capture(s);
    if (rc != GCOO_OK) return rc;

    gcoo_matrix* h = nullptr;
    rc = new_handle(m, k, nnz, p, dev_buf, &h, inside);
    if (rc != GCOO_OK) return rc;
    h->from_csr = true;
    char* base = h->base;
    char* scratch = inside ? base + L.persistent : reinterpret_cast<char*>(static_scratch_ptr);

    const int32_t* d_row_ptr = row_ptr;
    const int32_t* d_cols = col_idx;
    const float* d_vals = vals;
    HostStage stage;
    bool starts_given = false, narrow_cols = false;      // where the groups begin goes with the launch; the columns have 16 bits in the pinned buffer
    const size_t in_bytes = L.in_vals + (size_t)nnz * 4 - L.in_row_ptr;          // row_ptr, columns and values as they lie in the scratch area
    if (!src_on_device && in_bytes <= kStageBytes && stage.claim()) {
        // the caller may release its host arrays as soon as this call returns
        char* to = stage.ptr();
        std::memcpy(to, row_ptr, (size_t)(m + 1) * 4);
        const bool in_place = L.by_masks && h->has_rows();
        starts_given = in_place && L.plan.fused && g <= gcoo::kOrderHostGroups;
        narrow_cols = in_place && (starts_given || (!L.plan.fused && k <= 65536));
        if (nnz > 0) {
            if (narrow_cols) {
                uint16_t* narrow = reinterpret_cast<uint16_t*>(to + (L.in_cols - L.in_row_ptr));
                for (int64_t e = 0; e < nnz; ++e) narrow[e] = (uint16_t)col_idx[e];
            } else {
                std::memcpy(to + (L.in_cols - L.in_row_ptr), col_idx, (size_t)nnz * 4);
            }
            std::memcpy(to + (L.in_vals - L.in_row_ptr), vals, (size_t)nnz * 4);
        }
        if (in_place) {
            // every word of the input is read once: the kernel takes it from where it is
            void* seen = nullptr;
            hipError_t e = hipHostGetDevicePointer(&seen, to, 0);
            if (e != hipSuccess) { delete h; return hip_fail(e, "hipHostGetDevicePointer"); }
            to = static_cast<char*>(seen);
        } else {
            hipError_t e = hipMemcpyAsync(scratch + L.in_row_ptr, to, in_bytes, hipMemcpyHostToDevice, s);
            if (e != hipSuccess) { delete h; return hip_fail(e, "copy of the CSR input to the device"); }
            to = scratch + L.in_row_ptr;
        }
        d_row_ptr = reinterpret_cast<const int32_t*>(to);
        d_cols = reinterpret_cast<const int32_t*>(to + (L.in_cols - L.in_row_ptr));
        d_vals = reinterpret_cast<const float*>(to + (L.in_vals - L.in_row_ptr));
    } else if (!src_on_device) {
        int32_t* sp = reinterpret_cast<int32_t*>(scratch + L.in_row_ptr);
        int32_t* sc = reinterpret_cast<int32_t*>(scratch + L.in_cols);
        float* sv = reinterpret_cast<float*>(scratch + L.in_vals);
        hipError_t e = hipMemcpyAsync(sp, row_ptr, (size_t)(m + 1) * 4, hipMemcpyHostToDevice, s);
        if (e == hipSuccess && nnz > 0) e = hipMemcpyAsync(sc, col_idx, (size_t)nnz * 4, hipMemcpyHostToDevice, s);
        if (e == hipSuccess && nnz > 0) e = hipMemcpyAsync(sv, vals, (size_t)nnz * 4, hipMemcpyHostToDevice, s);
        // the caller may release its host arrays as soon as this call returns
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { delete h; return hip_fail(e, "copy of the CSR input to the device"); }
        d_row_ptr = sp; d_cols = sc; d_vals = sv;
    }

    bool marked = false;
    const int words = p <= 32 ? 1 : (p <= 64 ? 2 : 8);
    if (L.by_masks && L.plan.fused) {
        h->long_places = true;
        gcoo::OrderArgs o{};
        o.cols = d_cols; o.vals = d_vals; o.m = m; o.p = p; o.k = (int32_t)k; o.plan = L.plan; o.out = rows_out(h);
        o.dst_cols = h->cols(); o.dst_rows = h->rows(); o.dst_vals = h->values();
        o.row_ptr = d_row_ptr; o.nnz = (int32_t)nnz; o.g = g; o.gIdxes_out = h->gIdxes(); o.nnzPerGroup_out = h->nnzPerGroup();
        o.row_start_out = h->row_start(); o.flags_out = h->take_flags(); o.far = (bool)stage;
        if (starts_given) {
            // from the copy, which nobody else writes, and held inside the entries as the kernel holds what it reads itself
            const int32_t* copied = reinterpret_cast<const int32_t*>(stage.ptr());
            gcoo::GroupStarts starts;
            for (int64_t q = 0; q <= g; ++q) starts.at[q] = std::min(std::max(copied[q < g ? q * p : m], 0), (int32_t)nnz);
            auto order = L.plan.threads == 1024 ? (words == 1 ? gcoo::order_groups_host<1, 1024> : gcoo::order_groups_host<2, 1024>)
                                                : (words == 1 ? gcoo::order_groups_host<1, gcoo::kOrderThreads> : gcoo::order_groups_host<2, gcoo::kOrderThreads>);
            order<<<dim3((unsigned)g), dim3((unsigned)L.plan.threads), gcoo::order_lds_bytes(L.plan, words), s>>>(o, starts);
        } else {
        auto order = L.plan.threads == 1024 ? (words == 1 ? gcoo::order_groups<1, gcoo::kOrderFused, 1024> : (words == 2 ? gcoo::order_groups<2, gcoo::kOrderFused, 1024> : gcoo::order_groups<8, gcoo::kOrderFused, 1024>))
                                            : (words == 1 ? gcoo::order_groups<1, gcoo::kOrderFused> : (words == 2 ? gcoo::order_groups<2, gcoo::kOrderFused> : gcoo::order_groups<8, gcoo::kOrderFused>));
        order<<<dim3((unsigned)g), dim3((unsigned)L.plan.threads), gcoo::order_lds_bytes(L.plan, words), s>>>(o);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { delete h; return hip_fail(e, "order_groups"); }
    } else if (L.by_masks) {
        marked = L.band.h > 0 && !h->has_share;              // (the share schedule's builder uses the same scratch)
        gcoo::TakeArgs t{};
        t.row_ptr = d_row_ptr; t.cols = d_cols; t.vals = d_vals;
        t.m = m; t.g = g; t.lists = L.lists; t.p = p; t.nnz = (int32_t)nnz; t.k = (int32_t)k; t.plan = L.plan;
        t.gIdxes = h->gIdxes(); t.nnzPerGroup = h->nnzPerGroup(); t.row_start = h->row_start();
        t.row_cols = h->has_rows() ? h->row_cols() : nullptr; t.row_vals = h->row_vals();
        t.flags = h->take_flags(); t.splits = reinterpret_cast<int32_t*>(base + L.splits);
        t.bits = marked ? reinterpret_cast<uint32_t*>(scratch + L.tmp_cols) : nullptr;
        t.heavy = marked ? gcoo::band_heavy(nnz, L.lists) : INT32_MAX;
        t.zero_bad = h->bad_col();
        t.stats = h->has_sched ? stats : nullptr;
        const bool few = !stage && nnz / L.lists > 2048;
        (narrow_cols ? gcoo::take_rows<gcoo::kTakeHost16, 512> : (stage ? gcoo::take_rows<gcoo::kTakeHost, 512> : (few ? gcoo::take_rows<gcoo::kTakeDevice, 1024> : gcoo::take_rows<gcoo::kTakeDevice, 512>)))<<<
            dim3((unsigned)(L.lists + (h->has_sched ? 1 : 0))), dim3(few ? 1024 : 512), marked ? (size_t)((k + 31) / 32) * 4 : 0, s>>>(t);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { delete h; return hip_fail(e, "take_rows"); }
        gcoo::OrderArgs o{};
        o.row_start = h->row_start(); o.cols = h->has_rows() ? h->row_cols() : d_cols; o.vals = h->has_rows() ? h->row_vals() : d_vals;
        o.m = m; o.lists = L.lists; o.p = p; o.k = (int32_t)k; o.plan = L.plan; o.gIdxes = h->gIdxes(); o.flags = t.flags; o.splits = t.splits;
        o.out = rows_out(h); o.uneven = marked ? h->uneven() : nullptr; o.dst_cols = h->cols(); o.dst_rows = h->rows(); o.dst_vals = h->values();
        if (L.plan.both) {
            const gcoo::FillArgs f = fill_args(h, scratch, true);
            const int32_t lists = (int32_t)(gcoo::band_blocks(m, L.band.h) * gcoo::kBandWaves);
            const size_t fill_lds = gcoo::band_fill_lds(k, f.chunk, L.band.v), order_lds = gcoo::order_lds_bytes(L.plan, words);
            e = band_fill_lds_limit();
            if (e != hipSuccess) { delete h; return hip_fail(e, "order_and_fill"); }
            auto pick = [&](auto v) {
                constexpr int V = decltype(v)::value;
                return L.plan.keys ? (words == 1 ? gcoo::order_and_fill<1, gcoo::kOrderRanked, V> : gcoo::order_and_fill<2, gcoo::kOrderRanked, V>)
                                   : (words == 1 ? gcoo::order_and_fill<1, gcoo::kOrderMasks, V> : gcoo::order_and_fill<2, gcoo::kOrderMasks, V>);
            };
            (L.band.v == 4 ? pick(std::integral_constant<int, 4>{}) : pick(std::integral_constant<int, 2>{}))<<<
                dim3((unsigned)(lists + g * L.plan.parts)), dim3(gcoo::kBothThreads), fill_lds > order_lds ? fill_lds : order_lds, s>>>(o, f, lists);
        } else {
            auto order = L.plan.keys ? (words == 1 ? gcoo::order_groups<1, gcoo::kOrderRanked> : (words == 2 ? gcoo::order_groups<2, gcoo::kOrderRanked> : gcoo::order_groups<8, gcoo::kOrderRanked>))
                                   : (words == 1 ? gcoo::order_groups<1, gcoo::kOrderMasks> : (words == 2 ? gcoo::order_groups<2, gcoo::kOrderMasks> : gcoo::order_groups<8, gcoo::kOrderMasks>));
            order<<<dim3((unsigned)(g * L.plan.parts)), dim3(gcoo::kOrderThreads), gcoo::order_lds_bytes(L.plan, words), s>>>(o);
        }
        e = hipGetLastError();
        if (e != hipSuccess) { delete h; return hip_fail(e, "order_groups"); }
    } else
    // Algorithm 1, step 1: group index and counts straight from row_ptr (also writes the sentinel).
    {
        const unsigned blocks = (unsigned)(((h->has_rows() ? m : g) + 1 + 255) / 256) + 1u;     // the last one computes the statistics
        gcoo::group_index_from_row_ptr<<<dim3(blocks), dim3(256), 0, s>>>(d_row_ptr, m, p, g, (int32_t)nnz, h->gIdxes(), h->nnzPerGroup(),
                                                                         stats, h->bad_col(), h->has_rows() ? h->row_start() : nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { delete h; return hip_fail(e, "group_index_from_row_ptr"); }
    }
    // Algorithm 1, step 2: stable per-group radix sort on the column, 8 bits per pass, ping-pong
    // between the scratch triple and the final arrays so that the last pass lands in the latter.
    if (!L.by_masks && g > 0 && nnz > 0) {
        const int passes = radix_passes(k);
        int32_t* fin_c = h->cols(); int32_t* fin_r = h->rows(); float* fin_v = h->values();
        int32_t* tmp_c = reinterpret_cast<int32_t*>(scratch + L.tmp_cols);
        int32_t* tmp_r = reinterpret_cast<int32_t*>(scratch + L.tmp_rows);
        float* tmp_v = reinterpret_cast<float*>(scratch + L.tmp_vals);
        const int32_t* src_c = d_cols; const int32_t* src_r = nullptr; const float* src_v = d_vals;
        // Two passes and large groups: high digit first, then the low digit bucket by bucket (see the
        // kernel); otherwise low digit first, whole groups.
        const int64_t buckets = (k + 255) / 256;
        const bool high_first = passes == 2 && nnz / g >= 6000 && g * buckets <= 0x7fffffffLL;
        for (int pass = 0; pass < passes; ++pass) {
            const bool to_final = ((passes - 1 - pass) % 2) == 0;
            int32_t* dc = to_final ? fin_c : tmp_c;
            int32_t* dr = to_final ? fin_r : tmp_r;
            float* dv = to_final ? fin_v : tmp_v;
            const int shift = high_first ? 8 * (1 - pass) : 8 * pass;
            if (pass == 0)
                gcoo::sort_groups_by_col_digit<gcoo::kSortFirst, gcoo::kSortWaves><<<dim3((unsigned)g), dim3(gcoo::kSortWaves * gcoo::kWave), 0, s>>>(
                    h->gIdxes(), d_row_ptr, m, p, src_c, src_r, src_v, dc, dr, dv, shift, 0, (int32_t)k, h->bad_col(), rows_out(h));
            else if (high_first)
                gcoo::sort_groups_by_col_digit<gcoo::kSortNext, gcoo::kSortBucketWaves><<<dim3((unsigned)(g * buckets)), dim3(gcoo::kSortBucketWaves * gcoo::kWave), 0, s>>>(
                    h->gIdxes(), d_row_ptr, m, p, src_c, src_r, src_v, dc, dr, dv, shift, (int32_t)buckets, (int32_t)k, h->bad_col(), {});
            else
                gcoo::sort_groups_by_col_digit<gcoo::kSortNext, gcoo::kSortWaves><<<dim3((unsigned)g), dim3(gcoo::kSortWaves * gcoo::kWave), 0, s>>>(
                    h->gIdxes(), d_row_ptr, m, p, src_c, src_r, src_v, dc, dr, dv, shift, 0, (int32_t)k, h->bad_col(), {});
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) { delete h; return hip_fail(e, "sort_groups_by_col_digit"); }
            src_c = dc; src_r = dr; src_v = dv;
        }
    }
    if (stage) {
        // (what follows reads the entries in row order; with more than 64 rows per group, the copy on the device)
        hipError_t e = stage.release(s);
        if (e != hipSuccess) { delete h; return hip_fail(e, "hipEventRecord"); }
    }
    rc = launch_build_schedule(h, scratch, s, marked, L.by_masks && L.plan.both);
    if (rc != GCOO_OK) { delete h; return rc; }
    if (wants_inner(p)) {
        // the same entries once more, regrouped at kInnerP rows, from the CSR arrays on the device (a host input's
        // staged copy is still in this handle's scratch area, which the inner conversion does not touch)
        const size_t own = al(L.total);
        rc = from_csr(m, k, d_row_ptr, d_cols, d_vals, 1, nnz, kInnerP, base + own, dev_buf_bytes - own, stream, &h->inner,
                      static_scratch_ptr);
        if (rc != GCOO_OK) { delete h; return rc; }
    }
    *out = h;
    return GCOO_OK;
}

}  // namespace

extern "C" {

size_t gcoo_static_handle_bytes(int64_t m, int64_t k, int64_t nnz, int32_t p)
{
    if (!dims_ok(m, k, nnz, p) || nnz > kStaticMaxNnz) return 0;
    return total_bytes(m, k, nnz, p, false);
}

int gcoo_from_csr_device_static(int64_t m, int64_t k, int64_t nnz, const int32_t* row_ptr_dev, const int32_t* col_idx_dev,
                                const float* vals_dev, int32_t p, void* out_buf, size_t out_buf_bytes, void* stream,
                                gcoo_matrix** out)
{
    if (out) *out = nullptr;
    if (nnz < 0 || nnz > INT32_MAX) return GCOO_EINVAL;
    if (nnz > kStaticMaxNnz) return GCOO_ELIMIT;
    unsigned char* scratch = nullptr;
    int rc = static_scratch(&scratch);
    if (rc != GCOO_OK) return rc;
    return from_csr(m, k, row_ptr_dev, col_idx_dev, vals_dev, 1, nnz, p, out_buf, out_buf_bytes, stream, out, scratch);
}

int gcoo_from_csr(int64_t m, int64_t k, const int32_t* row_ptr, const int32_t* col_idx, const float* vals,
                  int src_on_device, int32_t p, void* dev_buf, size_t dev_buf_bytes, void* stream, gcoo_matrix** out)
{
    return from_csr(m, k, row_ptr, col_idx, vals, src_on_device, -1, p, dev_buf, dev_buf_bytes, stream, out);
}

int gcoo_from_csr_device(int64_t m, int64_t k, int64_t nnz, const int32_t* row_ptr_dev, const int32_t* col_idx_dev,
                         const float* vals_dev, int32_t p, void* dev_buf, size_t dev_buf_bytes, void* stream, gcoo_matrix** out)
{
    if (nnz < 0 || nnz > INT32_MAX) { if (out) *out = nullptr; return GCOO_EINVAL; }
    return from_csr(m, k, row_ptr_dev, col_idx_dev, vals_dev, 1, nnz, p, dev_buf, dev_buf_bytes, stream, out);
}

int gcoo_dense_nnz(int64_t m, int64_t k, const float* A_dev, int64_t lda, void* stream, int64_t* nnz)
{
    if (!nnz || m < 0 || k < 0 || lda < k || (m > 0 && k > 0 && !A_dev)) return GCOO_EINVAL;
    *nnz = 0;
    if (m == 0 || k == 0) return GCOO_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    HostSlot slot;
    int rc = slot.claim(s);
    if (rc != GCOO_OK) return rc;
    const int vw = dense_vec_width(A_dev, lda, k);
    const int64_t nblk = dense_blocks(k, vw);
    const int64_t items = (m + 15) / 16 * nblk;
    const dim3 grid((unsigned)(items < gcoo::kDenseWorkgroups ? items : gcoo::kDenseWorkgroups)), block(gcoo::kDenseThreads);
    if (vw == 4) gcoo::count_dense_total<4><<<grid, block, 0, s>>>(A_dev, lda, m, k, nblk, slot.ticket(), slot.host());
    else gcoo::count_dense_total<1><<<grid, block, 0, s>>>(A_dev, lda, m, k, nblk, slot.ticket(), slot.host());
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { slot.abandon(s); return hip_fail(e, "count_dense_total"); }
    unsigned long long got = 0;
    rc = slot.wait(s, &got);
    if (rc != GCOO_OK) return rc;
    *nnz = (int64_t)got;
    return GCOO_OK;
}

}  // extern "C"

namespace {

// Whether a count into a buffer of its own leaves a bit per element there, 64 bits per column of a group, so that the fill need not read A again.
// From 8 rows per group on they are a quarter of A or less.  Count, fill and schedules, reading A again and with the masks: 8000 x 8000, 0.5 %: p = 8 139 and
// 124 us, p = 64 132 and 95; 4000 x 4000, 20 %: p = 8 186 and 125 us, p = 64 353 and 206; 1000 x 1000: 1.00x to 1.23x.  With p = 4 they are half of A, and
// 8000 x 8000 takes 171 us instead of 161 at 0.5 % and 267 instead of 252 at 5 %.
bool dense_masks_wanted(int32_t p) { return p >= 8 && p <= 64; }

// Workgroups of fill_dense_groups() to a group: as many, up to four, as leave each no more entries than its LDS holds in row order, and 256 columns at least.  Each goes through all masks of its
// group, so that more are slower where one holds all (conversion with its count, us, 1, 2 and 4; entries per group in brackets: 4000 x 4000, 2 % (2560): 47.2 48.5 49.3; 5 % (6400): 58.5 54.6 55.1;
// 10 % (12800): 79.4 72.4 65.1; 6000 x 1000, 10 % (3200): 27.7 31.5 36.6; 500 x 4000, 20 % (25600): 84 62.7 48; 64 rows per group, 2000 x 2000, 2 % (2560): 30.2 27.2 28.4).
int32_t dense_groups_split(int64_t k, int64_t mean, int32_t p)
{
    const int64_t most = gcoo::dense_group_list(p), entries = mean + mean / 16;
    const int32_t split = entries <= most ? 1 : (entries <= 2 * most ? 2 : 4);
    return k <= 256 ? 1 : (k <= 512 && split > 2 ? 2 : split);
}
// Whether the fill, the order by rows and the bitmaps of the bands are one launch: where a workgroup has all columns of a group in its LDS, but not for many groups of a few rows each, which cost
// a workgroup of 1024 threads however little is in them (conversion with its count, us, three launches and one: 12000 x 3000, 1 %, 8 rows per group: 91 100; 20000 x 2000, 0.2 %, 16 rows: 57.1 57.6; 2000 x 2000, 1 %,
// 8 rows: 22.9 21.8).  Where there are bands it takes two launches off (308 shapes of 8 to 64 rows per group: 0.81 of the time; two of more than half of their cells filled 1.06 and 1.08).  Where there are none it takes one off and
// two workgroups to a compute unit are one round: beyond that only groups of a thousand entries in 200 columns (us, two launches and one, 32 rows per group: 60000 x 64, 16 and 31 % (160 and 640 per group): 43.2 48.5, 52.7 62.6;
// 200000 x 256, 0.5 %: 110 124; 60000 x 1024, 0.1 %: 73 77; 40000 x 300, 15 % (1440): 55 53, 30 %: 71 61; the group in two parts, 60 % (5760, 24 rows): 135 192).  And a thread goes through all bits of its four columns,
// so not narrow matrices of which most is filled, nor groups of more than 32 rows whose entries do not fit the list, while their columns are one part or hardly two (200 x 64, all filled: 1.04 and 1.06 of the time at 24 and 32 rows per group,
// 1.35 to 1.56 at 64; 64 rows, 4000 x 128, 31 %: 34.5 42.2; 256 columns, 35 to 100 %: 1.1 to 1.7; 512: 0.84 to 1).
bool dense_groups_wanted(int64_t m, int64_t k, int64_t nnz, int32_t p, BandPlan band)
{
    const int64_t g = (m + p - 1) / p, mean = nnz / g;
    if (k > gcoo::kDenseWindow || (p < 24 && g > 512)) return false;
    // a group lies in two blocks at the most, and the bitmaps go where the lists' would, into three words per entry
    if (band.h > 0) return gcoo::kBandWaves * band.h >= p && (g + gcoo::band_blocks(m, band.h)) * ((k + 31) / 32) <= 3 * nnz;
    const int32_t split = dense_groups_split(k, mean, p);
    if (g * split > 512 && (split > 1 || k < 200 || mean < 1000)) return false;
    return !(k <= 64 && mean > 24 * k) && !(p > 32 && k <= 300 && mean + mean / 16 > gcoo::dense_group_list(p));
}

// The counts of a dense matrix, at the places where a matrix buffer has them (offsets that do not depend on nnz).
// `masks`: a buffer that holds them as well, behind the others.
gcoo::DenseCounts dense_counts(void* buf, const Layout& L, bool masks)
{
    char* base = static_cast<char*>(buf);
    return {reinterpret_cast<gcoo::Handed<int32_t>*>(base + L.blk), reinterpret_cast<int32_t*>(base + L.gIdxes),
            reinterpret_cast<int32_t*>(base + L.nnzPerGroup), reinterpret_cast<unsigned long long*>(base + L.counter),
            masks ? reinterpret_cast<uint64_t*>(base + L.values) : nullptr};
}

// Step 1 of Algorithm 1.  `host` receives the sum, or is null.
int launch_dense_count(int64_t m, int64_t k, const float* A_dev, int64_t lda, int32_t p, void* buf, bool masks, gcoo::DenseTicket ticket,
                       unsigned long long* host, hipStream_t s)
{
    const int64_t g = (m + p - 1) / p;
    const int vw = dense_vec_width(A_dev, lda, k);
    const int64_t nblk = dense_blocks(k, vw);
    // one workgroup per (group, column block) fills; a band holds fewer than 2^31 elements so that
    // 32-bit counts cannot wrap before the total is checked
    if (nblk > 0 && g > 0x7fffffffLL / nblk) return GCOO_EINVAL;
    if ((int64_t)p * k > INT32_MAX) return GCOO_EINVAL;
    const gcoo::DenseCounts out = dense_counts(buf, make_layout(m, k, 0, g, p), masks);
    const int64_t items = g * nblk;
    const dim3 grid((unsigned)(items < 1 ? 1 : (items < gcoo::kDenseWorkgroups ? items : gcoo::kDenseWorkgroups))), block(gcoo::kDenseThreads);
    (vw == 4 ? (masks ? gcoo::count_dense_blocks<4, true> : gcoo::count_dense_blocks<4, false>)
             : (masks ? gcoo::count_dense_blocks<1, true> : gcoo::count_dense_blocks<1, false>))<<<grid, block, 0, s>>>(
        A_dev, lda, m, k, p, nblk, g, out, ticket, host);
    HIP_TRY(hipGetLastError());
    return GCOO_OK;
}

// The same, and the wait for its sum.  `own_buf`: counts only, the matrix gets a buffer of its own.  In the buffer of the matrix (gcoo_from_dense()) the call waits for
// the stream without a look: that it synchronises is its description, and a caller may read in its status whether the work before it went well, which a number
// that has come does not say.
int count_dense(int64_t m, int64_t k, const float* A_dev, int64_t lda, int32_t p, void* buf, bool own_buf, hipStream_t s, int64_t* nnz)
{
    HostSlot slot;
    int rc = slot.claim(s);
    if (rc != GCOO_OK) return rc;
    rc = launch_dense_count(m, k, A_dev, lda, p, buf, own_buf && dense_masks_wanted(p), slot.ticket(), slot.host(), s);
    if (rc == GCOO_EHIP) slot.abandon(s);
    if (rc != GCOO_OK) return rc;
    unsigned long long total = 0;
    rc = own_buf ? slot.look(s, &total) : slot.wait(s, &total);
    if (rc != GCOO_OK) return rc;
    if (total > (unsigned long long)INT32_MAX) return GCOO_EINVAL;
    *nnz = (int64_t)total;
    return GCOO_OK;
}

int from_dense_counted(int64_t m, int64_t k, int64_t nnz, const float* A_dev, int64_t lda, int32_t p, const void* counts, void* dev_buf,
                       size_t dev_buf_bytes, void* stream, gcoo_matrix** out)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t g = (m + p - 1) / p;
    if (dev_buf_bytes < total_bytes(m, k, nnz, p, true)) return GCOO_ENOMEM;
    gcoo_matrix* h = nullptr;
    int rc = new_handle(m, k, nnz, p, dev_buf, &h);
    if (rc != GCOO_OK) return rc;
    const int vw = dense_vec_width(A_dev, lda, k);
    const int64_t nblk = dense_blocks(k, vw);
    const bool masks = counts != dev_buf && dense_masks_wanted(p);        // (in a buffer of its own the matrix lies where they would)
    const gcoo::DenseCounts from = dense_counts(const_cast<void*>(counts), h->L, masks), to = dense_counts(dev_buf, h->L, false);
    const bool grouped = masks && g > 0 && k > 0 && dense_groups_wanted(m, k, nnz, p, h->L.band) && !h->has_share;
    // Groups of more than 64 rows: the regrouped copy is counted on the device alone, behind the fill, which clears its ticket.
    const size_t own = al(h->L.total);
    char* inner_buf = nullptr;
    unsigned long long* inner_ticket = nullptr;
    if (wants_inner(p)) {
        inner_buf = h->base + own;
        inner_ticket = reinterpret_cast<unsigned long long*>(inner_buf + make_layout(m, k, 0, (m + kInnerP - 1) / kInnerP, kInnerP).counter + kTicketAt);
    }
    {
        const dim3 grid((unsigned)(g * nblk > 0 ? g * nblk : 1)), block(gcoo::kDenseThreads);
        const bool small = p <= 64;
        if (grouped) {
            const bool band = h->L.band.h > 0;
            h->long_places = !band;
            const int32_t split = dense_groups_split(k, nnz / g, p);
            (split > 1 ? (p <= 32 ? gcoo::fill_dense_groups<32, true> : gcoo::fill_dense_groups<64, true>) : (p <= 32 ? gcoo::fill_dense_groups<32, false> : gcoo::fill_dense_groups<64, false>))<<<dim3((unsigned)(g * split)), dim3(gcoo::kDenseGroupThreads), 0, s>>>(
                A_dev, lda, m, k, p, g, from, to, h->bad_col(), h->values(), h->rows(), h->cols(), rows_out(h), !band,
                band ? reinterpret_cast<uint32_t*>(h->base + h->L.persistent + h->L.tmp_cols) : nullptr, gcoo::kBandWaves * h->L.band.h, split);
        } else if (masks)
            (vw == 4 ? gcoo::fill_dense_masked<4> : gcoo::fill_dense_masked<1>)<<<grid, block, 0, s>>>(
                A_dev, lda, k, p, nblk, g, from, to, h->bad_col(), h->values(), h->rows(), h->cols());
        else (vw == 4 ? (small ? gcoo::fill_dense_blocks<4, true> : gcoo::fill_dense_blocks<4, false>)
                 : (small ? gcoo::fill_dense_blocks<1, true> : gcoo::fill_dense_blocks<1, false>))<<<grid, block, 0, s>>>(
            A_dev, lda, m, k, p, nblk, g, from, to, h->bad_col(), inner_ticket, h->values(), h->rows(), h->cols());
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { delete h; return hip_fail(e, "fill_dense_blocks"); }
    }
    if (g > 0 && h->has_rows() && !grouped) {
        gcoo::sort_groups_by_col_digit<gcoo::kSortByRow, gcoo::kSortWaves><<<dim3((unsigned)g), dim3(gcoo::kSortWaves * gcoo::kWave), 0, s>>>(
            h->gIdxes(), nullptr, m, p, h->cols(), h->rows(), h->values(), h->row_cols(), nullptr, h->row_vals(), 0, 0, (int32_t)k,
            nullptr, rows_out(h));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { delete h; return hip_fail(e, "sort_groups_by_col_digit"); }
    }
    rc = launch_build_schedule(h, h->base + h->L.persistent, s, grouped && h->L.band.h > 0, false, grouped);
    if (rc != GCOO_OK) { delete h; return rc; }
    if (inner_buf) {
        rc = launch_dense_count(m, k, A_dev, lda, kInnerP, inner_buf, false, {inner_ticket, 1}, nullptr, s);
        if (rc == GCOO_OK)
            rc = from_dense_counted(m, k, nnz, A_dev, lda, kInnerP, inner_buf, inner_buf, dev_buf_bytes - own, stream, &h->inner);
        if (rc != GCOO_OK) { delete h; return rc; }
    }
    *out = h;
    return GCOO_OK;
}

bool dense_args_ok(int64_t m, int64_t k, const float* A_dev, int64_t lda, int32_t p, const void* buf)
{
    return buf && dims_ok(m, k, 0, p) && lda >= k && (m == 0 || k == 0 || A_dev) && reinterpret_cast<uintptr_t>(buf) % kAlign == 0;
}

}  // namespace

extern "C" {

size_t gcoo_dense_count_bytes(int64_t m, int64_t k, int32_t p)
{
    if (!dims_ok(m, k, 0, p)) return 0;
    const int64_t g = (m + p - 1) / p;
    return make_layout(m, k, 0, g, p).values + (dense_masks_wanted(p) ? al((size_t)g * k * 8) : 0);
}

int gcoo_dense_count(int64_t m, int64_t k, const float* A_dev, int64_t lda, int32_t p, void* count_buf, size_t count_buf_bytes,
                     void* stream, int64_t* nnz)
{
    if (!nnz) return GCOO_EINVAL;
    *nnz = 0;
    if (!dense_args_ok(m, k, A_dev, lda, p, count_buf)) return GCOO_EINVAL;
    if (count_buf_bytes < gcoo_dense_count_bytes(m, k, p)) return GCOO_ENOMEM;
    return count_dense(m, k, A_dev, lda, p, count_buf, true, static_cast<hipStream_t>(stream), nnz);
}

int gcoo_from_dense_counted(int64_t m, int64_t k, int64_t nnz, const float* A_dev, int64_t lda, int32_t p, const void* count_buf,
                            void* dev_buf, size_t dev_buf_bytes, void* stream, gcoo_matrix** out)
{
    const PolicyOfCall policy_of_call;
    if (!out) return GCOO_EINVAL;
    *out = nullptr;
    if (!dense_args_ok(m, k, A_dev, lda, p, dev_buf) || !count_buf || reinterpret_cast<uintptr_t>(count_buf) % kAlign) return GCOO_EINVAL;
    if (!dims_ok(m, k, nnz, p) || nnz > m * k) return GCOO_EINVAL;
    return from_dense_counted(m, k, nnz, A_dev, lda, p, count_buf, dev_buf, dev_buf_bytes, stream, out);
}

int gcoo_from_dense(int64_t m, int64_t k, const float* A_dev, int64_t lda, int32_t p, void* dev_buf, size_t dev_buf_bytes,
                    void* stream, gcoo_matrix** out)
{
    const PolicyOfCall policy_of_call;
    if (!out) return GCOO_EINVAL;
    *out = nullptr;
    if (!dense_args_ok(m, k, A_dev, lda, p, dev_buf)) return GCOO_EINVAL;
    // The counts sit at the front of the buffer at offsets that do not depend on nnz, so step 1 can run before the buffer size for
    // this nnz is checked.
    if (dev_buf_bytes < make_layout(m, k, 0, (m + p - 1) / p, p).total) return GCOO_ENOMEM;
    int64_t nnz = 0;
    const int rc = count_dense(m, k, A_dev, lda, p, dev_buf, false, static_cast<hipStream_t>(stream), &nnz);
    if (rc != GCOO_OK) return rc;
    return from_dense_counted(m, k, nnz, A_dev, lda, p, dev_buf, dev_buf, dev_buf_bytes, stream, out);
}

}  // extern "C"

namespace {

struct Shape {
    bool al4;          // N, both leading dimensions and both base addresses fit 16-byte accesses: what the
                       // workgroup-shared kernel's loads straight to LDS need
    bool b16;          // B begins at a multiple of 16 bytes
    bool wide_pitch;   // row pitch of B in bytes does not fit 32 bits: LDS variant only
    int64_t N;
};

Shape shape_of(const float* B, int64_t ldb, int64_t N, const float* C, int64_t ldc)
{
    const uintptr_t pb = reinterpret_cast<uintptr_t>(B), pc = reinterpret_cast<uintptr_t>(C);
    Shape s;
    s.al4 = (N % 4 == 0) && (ldb % 4 == 0) && (ldc % 4 == 0) && (pb % 16 == 0) && (pc % 16 == 0);
    s.b16 = pb % 16 == 0;
    s.wide_pitch = ldb > 0x3fffffffLL;
    s.N = N;
    return s;
}

// Instance of the register kernel that serves this p and N: its columns per lane, 0 if none does;
// kTallInstance for four columns per lane with the tall accumulator file (33 <= p <= 38).  The instances
// take any N of at least their columns per lane and any leading dimensions and base addresses: the one lane that
// would reach beyond N computes the last columns of the row instead (lane_cols() in gcoo_spdm_kernels.hpp), and
// rows that are aligned to 4 bytes only are read and written with unaligned 16-byte accesses.
constexpr int kTallInstance = 38;
int sched_width(int32_t p, const Shape& sh)
{
    if (sh.wide_pitch) return 0;
    if (p <= 32 && sh.N >= 4) return 4;
    if (p <= 38 && sh.N >= 4) return kTallInstance;
    if (p <= 64 && sh.N >= 2) return 2;
    // There is no one-column-per-lane instance (65 <= p <= 128, or N = 1): a run of one on an 8000 x 8000
    // matrix with p = 128 ended in a GPU memory fault whose cause was never found, and it was taken out of
    // the build.  Such calls are multiplied row by row (automatic choice) or get GCOO_EINVAL (explicit GCOO_VARIANT_REG).
    return 0;
}

}  // namespace

namespace gcoo {
hipError_t launch_spdm_sched(int V, const SpdmArgs& a, hipStream_t s)
{
    if (V == 4) return launch_spdm_sched_v4(a, s);
    if (V == 38) return launch_spdm_sched_v4_tall(a, s);
    if (V == 2) return launch_spdm_sched_v2(a, s);
    return hipErrorInvalidValue;
}
}  // namespace gcoo

namespace {

bool share_operands_ok(const gcoo_matrix* A, const Shape& sh, int64_t ldb)
{
    // (the workgroup-shared kernel keeps byte offsets into B in 32 bits, each up to 3072 above the place it stands for; the limit of the
    // sixteen-wave kernel is the same)
    return sh.al4 && (uint64_t)A->k * (uint64_t)ldb * 4u <= gcoo::kRowsMaxBytes;
}

bool band_operands_ok(const gcoo_matrix* A, const Shape& sh, int64_t ldb)
{
    const bool aligned = sh.N % 4 == 0 && ldb % 4 == 0 && sh.b16;
    return (aligned || sh.N >= 64 * A->L.band.v) && (uint64_t)A->k * (uint64_t)ldb * 4u <= gcoo::kRowsMaxBytes;
}

// Row by row before the register kernel, for a handle that carries the run schedule: up to about 30 entries per row (n = 4000: level at
// 1.2 %, n = 8000: 0.45 %), and well above a hundred where the groups' items fill less than half of the 2048 wave slots.
bool rows_preferred(const gcoo_matrix* A, int64_t N)
{
    if (A->nnz <= 28 * A->m) return true;
    return A->g * ((N + 255) / 256) <= 1024 && A->nnz <= 128 * A->m;
}

int check_spdm_args(const gcoo_matrix* A, const float* B, int64_t ldb, int64_t N, const float* C, int64_t ldc)
{
    if (!A || N < 0 || ldb < N || ldc < N || N > INT32_MAX) return GCOO_EINVAL;
    if (N > 0 && A->m > 0 && !C) return GCOO_EINVAL;
    if (N > 0 && A->nnz > 0 && !B) return GCOO_EINVAL;
    return GCOO_OK;
}

}  // namespace

extern "C" {

int gcoo_spdm_pick(const gcoo_matrix* A, const float* B_dev, int64_t ldb, int64_t N, const float* C_dev, int64_t ldc)
{
    int rc = check_spdm_args(A, B_dev, ldb, N, C_dev, ldc);
    if (rc != GCOO_OK) return rc;
    if (A->inner) A = A->inner;        // groups taller than 64 rows: the fast kernels run on the regrouped copy
    const Shape sh = shape_of(B_dev, ldb, N, C_dev, ldc);
    // the workgroup-shared kernel wants enough workgroups to occupy the chip (one per 8p rows and 256 columns),
    // and below 9000 columns its margin over the register kernel does not survive a last round that is mostly idle
    const int64_t items = A->share_nq() * ((N + 255) / 256);
    if (A->share_preferred && share_operands_ok(A, sh, ldb) && items >= 192 && (A->k >= 9000 || fill_of_rounds(items) >= 0.8))
        return GCOO_VARIANT_SHARE;
    return (A->has_rows() && sched_width(A->p, sh)) ? GCOO_VARIANT_REG : GCOO_VARIANT_LDS;
}

}  // extern "C"

namespace {

// The kernel that a product runs (GCOO_KERNEL_*), or GCOO_EINVAL.  The arguments have passed check_spdm_args().  *M becomes the copy
// regrouped at kInnerP rows where the product is made with that.
int kernel_of_product(const gcoo_matrix** M, const Shape& sh, const float* B_dev, int64_t ldb, const float* C_dev, int64_t ldc, int variant)
{
    const gcoo_matrix* A = *M;
    const int64_t N = sh.N;
    if (variant < GCOO_VARIANT_AUTO || variant > GCOO_VARIANT_SHARE) return GCOO_EINVAL;
    if (A->m == 0 || N == 0) return GCOO_KERNEL_NONE;
    const bool automatic = variant == GCOO_VARIANT_AUTO;
    if (automatic) variant = gcoo_spdm_pick(A, B_dev, ldb, N, C_dev, ldc);
    // The automatic choice leaves the LDS kernel a row pitch of B that the others do not hold in 32 bits, and a matrix without columns, which
    // the row-by-row kernel does not take.
    if (automatic ? A->k < 1 || (variant == GCOO_VARIANT_LDS && sh.wide_pitch) : variant == GCOO_VARIANT_LDS) return GCOO_KERNEL_LDS;
    if (A->inner) *M = A = A->inner;   // the schedules of the other kernels belong to the regrouped copy
    if (automatic && A->has_rows()) {
        const bool lines = ldb % 32 == 0 && reinterpret_cast<uintptr_t>(B_dev) % 128 == 0;
        if (A->L.band.h > 0 && band_operands_ok(A, sh, ldb) &&
            band_time(A->m, A->k, A->nnz, N, A->L.band, lines) < no_schedule_time(A->m, A->k, A->nnz, N, lines))
            return GCOO_KERNEL_BAND;
        if (!A->has_sched || rows_preferred(A, N) || sched_width(A->p, sh) == 0) return GCOO_KERNEL_ROWS;     // (0: fewer columns than the register kernel serves)
    }
    if (variant == GCOO_VARIANT_SHARE) {
        if (!share_operands_ok(A, sh, ldb)) return GCOO_EINVAL;
        if (A->has_share) return GCOO_KERNEL_SHARE;
        return A->share_preferred && band_operands_ok(A, sh, ldb) ? GCOO_KERNEL_BAND : GCOO_EINVAL;
    }
    if (sched_width(A->p, sh) == 0 || !A->has_rows()) return GCOO_EINVAL;
    if (A->k < 1) return GCOO_KERNEL_LDS;
    return A->has_sched ? GCOO_KERNEL_SCHED : GCOO_KERNEL_ROWS;
}

}  // namespace

extern "C" {

int gcoo_spdm_kernel(const gcoo_matrix* A, const float* B_dev, int64_t ldb, int64_t N, const float* C_dev, int64_t ldc, int variant)
{
    const int rc = check_spdm_args(A, B_dev, ldb, N, C_dev, ldc);
    if (rc != GCOO_OK) return rc;
    return kernel_of_product(&A, shape_of(B_dev, ldb, N, C_dev, ldc), B_dev, ldb, C_dev, ldc, variant);
}

int gcoo_spdm_variant(const gcoo_matrix* A, const float* B_dev, int64_t ldb, int64_t N, float* C_dev, int64_t ldc,
                      void* stream, int variant)
{
    const int rc = check_spdm_args(A, B_dev, ldb, N, C_dev, ldc);
    if (rc != GCOO_OK) return rc;
    const Shape sh = shape_of(B_dev, ldb, N, C_dev, ldc);
    const int kernel = kernel_of_product(&A, sh, B_dev, ldb, C_dev, ldc, variant);
    if (kernel <= GCOO_KERNEL_NONE) return kernel;
    hipStream_t s = static_cast<hipStream_t>(stream);

    if (kernel == GCOO_KERNEL_LDS) {
        const int64_t tiles = (N + 63) / 64;
        const int64_t total = A->g * tiles;
        if (total > 0x7fffffffLL) return GCOO_EINVAL;
        const size_t smem = (size_t)A->p * 64 * sizeof(float);
        gcoo::spdm_lds<<<dim3((unsigned)total), dim3(64), smem, s>>>(A->values(), A->rows(), A->cols(), A->gIdxes(), A->m,
                                                                     A->p, B_dev, ldb, N, C_dev, ldc, A->g);
        HIP_TRY(hipGetLastError());
        return GCOO_OK;
    }
    if (kernel == GCOO_KERNEL_ROWS || kernel == GCOO_KERNEL_BAND) {
        gcoo::RowsArgs rows{A->row_start(), A->row_cols(), A->row_vals(), A->m, A->k, A->nnz, B_dev, ldb, N, C_dev, ldc,
                            A->long_rows(), A->long_count(), gcoo::rows_long(A->m, A->nnz), long_room(A->m, A->nnz), 0};
        if (A->long_places) {
            // no places are looked at where only a row that repeats columns could be long
            const bool some = A->k > rows.long_row;
            rows.long_count = nullptr;
            rows.long_room = some ? (int32_t)(A->nnz / rows.long_row) : 0;
            if (!some) rows.long_row = INT32_MAX;
        }
        if (kernel == GCOO_KERNEL_ROWS) {
            const bool lines = ldb % 32 == 0 && reinterpret_cast<uintptr_t>(B_dev) % 128 == 0, reach = (uint64_t)A->k * (uint64_t)ldb * 4u <= gcoo::kRowsMaxBytes;
            const TilePlan& plan = tile_plan(A->m, A->k, A->nnz, N);
            hipError_t e = reach && plan.preferred[lines] ? gcoo::launch_spdm_rows_tile(rows, plan.row_wgs, plan.whole, s) : gcoo::launch_spdm_rows(rows, !A->from_csr, s);
            return e == hipSuccess ? GCOO_OK : hip_fail(e, "spdm_rows launch");
        }
        gcoo::BandArgs a{A->band_head(), A->band_units(), A->band_first(), A->band_count(), (int32_t)gcoo::band_blocks(A->m, A->L.band.h), A->L.band.h, A->L.band.v,
                         0, 0, A->uneven(), gcoo::band_head_stride(A->k, A->L.band.v), A->m, A->k, B_dev, ldb, N, C_dev, ldc};
        hipError_t e = gcoo::launch_spdm_band(a, rows, s);
        return e == hipSuccess ? GCOO_OK : hip_fail(e, "spdm_band launch");
    }
    if (kernel == GCOO_KERNEL_SHARE) {
        gcoo::ShareArgs a{A->share_hdr(), A->share_blocks(), A->share_sbase(), A->share_ucols(), A->share_ucount(), A->gIdxes(),
                          A->m, A->p, A->g, A->share_nq(), B_dev, ldb, N, C_dev, ldc};
        hipError_t e = gcoo::launch_spdm_share(a, s);
        return e == hipSuccess ? GCOO_OK : hip_fail(e, "spdm_share launch");
    }
    const int V = sched_width(A->p, sh);
    const int cols_per_lane = V == kTallInstance ? 4 : V;
    // Heavy groups are shared by a workgroup in the standard instances only, and only a launch of few
    // items can have any: then the kernels decide group by group, from the statistics on the device.
    const bool heavy = V != kTallInstance && gcoo::sched_heavy_possible(A->nnz, A->g, (N + 64 * cols_per_lane - 1) / (64 * cols_per_lane));
    gcoo::SpdmArgs a{A->sched_hdr(), A->sched(), A->gIdxes(), A->m, A->p, A->g, A->nw, B_dev, ldb, N, C_dev, ldc,
                     A->nnz, heavy ? A->stats() : nullptr, (heavy && A->has_order()) ? A->order() : nullptr};
    hipError_t e = gcoo::launch_spdm_sched(V, a, s);
    if (e != hipSuccess) return hip_fail(e, "spdm_sched launch");
    return GCOO_OK;
}

int gcoo_spdm(const gcoo_matrix* A, const float* B_dev, int64_t ldb, int64_t N, float* C_dev, int64_t ldc, void* stream)
{
    return gcoo_spdm_variant(A, B_dev, ldb, N, C_dev, ldc, stream, GCOO_VARIANT_AUTO);
}

int gcoo_free(gcoo_matrix* A)
{
    delete A;
    return GCOO_OK;
}

int gcoo_info(const gcoo_matrix* A, int64_t* m, int64_t* k, int64_t* nnz, int32_t* p, int64_t* g)
{
    if (!A) return GCOO_EINVAL;
    if (m) *m = A->m;
    if (k) *k = A->k;
    if (nnz) *nnz = A->nnz;
    if (p) *p = A->p;
    if (g) *g = A->g;
    return GCOO_OK;
}

int gcoo_export(const gcoo_matrix* A, float* values, int32_t* rows, int32_t* cols, int64_t* gIdxes, int32_t* nnzPerGroup,
                void* stream)
{
    if (!A) return GCOO_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t n4 = (size_t)A->nnz * 4;
    if (values && n4) HIP_TRY(hipMemcpyAsync(values, A->values(), n4, hipMemcpyDeviceToHost, s));
    if (rows && n4) HIP_TRY(hipMemcpyAsync(rows, A->rows(), n4, hipMemcpyDeviceToHost, s));
    if (cols && n4) HIP_TRY(hipMemcpyAsync(cols, A->cols(), n4, hipMemcpyDeviceToHost, s));
    if (nnzPerGroup && A->g) HIP_TRY(hipMemcpyAsync(nnzPerGroup, A->nnzPerGroup(), (size_t)A->g * 4, hipMemcpyDeviceToHost, s));
    // columns out of range: one word, or one per list of rows that the conversion took
    const bool lists = A->from_csr && A->L.by_masks;
    const size_t n_bad = lists ? (size_t)A->L.lists : 1;
    std::unique_ptr<int32_t[]> narrow(gIdxes ? new (std::nothrow) int32_t[(size_t)A->g + 1] : nullptr);
    std::unique_ptr<uint32_t[]> bad(new (std::nothrow) uint32_t[n_bad]);
    if ((gIdxes && !narrow) || !bad) return GCOO_ENOMEM;
    if (gIdxes) HIP_TRY(hipMemcpyAsync(narrow.get(), A->gIdxes(), (size_t)(A->g + 1) * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(bad.get(), lists ? A->take_flags() : A->bad_col(), n_bad * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (gIdxes)
        for (int64_t i = 0; i <= A->g; ++i) gIdxes[i] = narrow[i];
    uint32_t any = 0;
    for (size_t i = 0; i < n_bad; ++i) any |= bad[i] & (lists ? gcoo::kBadColumn : ~0u);
    return any ? GCOO_EBOUNDS : GCOO_OK;
}

int gcoo_export_share(const gcoo_matrix* A, uint32_t* hdr, uint32_t* blocks, int32_t* sbase, int32_t* ucount, int32_t* ucols,
                      int64_t* hdr_words, int64_t* block_count, void* stream)
{
    if (!A) return GCOO_EINVAL;
    if (!A->has_share) {
        if (!A->share_preferred) return GCOO_EINVAL;
        if (hdr_words) *hdr_words = 0;
        if (block_count) *block_count = 0;
        return GCOO_OK;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t hw = gcoo::share_hdr_words(A->nnz, A->g), nb = gcoo::share_stream_blocks(A->nnz, A->g, A->k);
    if (hdr_words) *hdr_words = hw;
    if (block_count) *block_count = nb;
    if (hdr) HIP_TRY(hipMemcpyAsync(hdr, A->share_hdr(), (size_t)hw * 4, hipMemcpyDeviceToHost, s));
    if (blocks) HIP_TRY(hipMemcpyAsync(blocks, A->share_blocks(), (size_t)nb * gcoo::kShareBlockWords * 4, hipMemcpyDeviceToHost, s));
    if (sbase) HIP_TRY(hipMemcpyAsync(sbase, A->share_sbase(), (size_t)A->share_nq() * gcoo::kShareW * 4, hipMemcpyDeviceToHost, s));
    if (ucount) HIP_TRY(hipMemcpyAsync(ucount, A->share_ucount(), (size_t)A->share_nq() * 4, hipMemcpyDeviceToHost, s));
    if (ucols && A->nnz) HIP_TRY(hipMemcpyAsync(ucols, A->share_ucols(), (size_t)A->nnz * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return GCOO_OK;
}

const char* gcoo_strerror(int status)
{
    switch (status) {
        case GCOO_OK: return "ok";
        case GCOO_EINVAL: return "invalid argument";
        case GCOO_EBOUNDS: return "malformed CSR input (row_ptr not non-decreasing from 0, or column out of range)";
        case GCOO_ENOMEM: return "device buffer too small (see gcoo_device_bytes) or host allocation failed";
        case GCOO_EHIP: return "HIP runtime error (see gcoo_last_hip_error)";
        case GCOO_ELIMIT: return "input larger than the fixed scratch of gcoo_from_csr_device_static (at most 2097152 stored entries)";
        default: return "unknown status";
    }
}

const char* gcoo_last_hip_error(void) { return g_hip_error.c_str(); }

}  // extern "C"
