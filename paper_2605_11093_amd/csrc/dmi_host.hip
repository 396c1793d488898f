// Host runtime of the capture-and-stage library: ring ownership, policy gate and
// admission (paper section 4.4), kernel launches for dmi_observe (section 4.2), the
// drain stage and pinned host ring (section 4.3), and the core of the C ABI of include/dmi.h
// (replayable steps: dmi_step.hip; exporter: dmi_exporter.hip).
#include "dmi_ring.h"

using namespace dmi;
using namespace dmi::host;

namespace dmi {
namespace host {

static thread_local std::string g_err;

dmi_status_t fail(dmi_status_t code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

const char *last_error_cstr() { return g_err.c_str(); }

}  // namespace host
}  // namespace dmi

namespace dmi {
namespace host {

void atomic_max(std::atomic<uint64_t> &a, uint64_t v)
{
    uint64_t cur = a.load(std::memory_order_relaxed);
    while (cur < v && !a.compare_exchange_weak(cur, v, std::memory_order_relaxed)) {}
}

const void *this_thread()
{
    static thread_local char here;
    return &here;
}

void note_producer(dmi_ring *r, void *stream)
{
    r->producer.store(this_thread(), std::memory_order_relaxed);
    r->last_stream.store(stream, std::memory_order_release);
}

// Whether `s` is being captured.  The runtime may decline to say (of the null stream, while another thread captures
// one that waits for it); the error it leaves is cleared, or the thread's next launch would be reported as failed.
bool capture_status(hipStream_t s, hipStreamCaptureStatus *status)
{
    if (hipStreamIsCapturing(s, status) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Record an event behind everything launched so far (no-op if that is already covered).
// If the host cannot tell what those launches added (drop-newest, keep vectors), the
// newest launch's commit slot is fetched into the pinned mirror in front of the event.
// Both go onto the producer's own stream: a launch on a second hardware queue that waits
// for an event of this one slows every dispatch here by a microsecond or so while it
// waits, far more than a small launch every sixteenth capture costs in line.
dmi_status_t record_probe(dmi_ring *r)
{
    std::lock_guard<std::mutex> lk(r->pmu);
    const uint64_t launched = r->next_seq.load(std::memory_order_acquire);
    if (launched <= r->probed_upto) return DMI_OK;
    hipEvent_t ev;
    if (r->probe_pool.empty()) HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    else { ev = r->probe_pool.back(); r->probe_pool.pop_back(); }
    hipStream_t us = (hipStream_t)r->last_stream.load(std::memory_order_acquire);
    const bool fetch = !r->window_exact;
    if (fetch) {
        const uint32_t slot = (uint32_t)((launched - 1u) % kCommitSlots);
        HIP_TRY(launch_fetch_slot(&r->dctrl->slots[slot], r->hslots_dev + slot, us));
    }
    HIP_TRY(hipEventRecord(ev, us));
    r->probes.push_back({ev, DrainNote(), launched, r->launches.load(std::memory_order_relaxed), fetch, r->window, ++r->probes_made, us,
                         hipSuccess});
    r->window = Delta();
    r->window_exact = true;
    r->probed_upto = launched;
    return DMI_OK;
}

// The same where a drain kernel that says itself when it is over has gone behind everything launched so far.  Caller
// has seen that the host can tell what those launches add.
static uint64_t probe_by_drain(dmi_ring *r, const DrainNote &note, hipStream_t us)
{
    std::lock_guard<std::mutex> lk(r->pmu);
    const uint64_t launched = r->next_seq.load(std::memory_order_acquire);
    r->probes.push_back({nullptr, note, launched, r->launches.load(std::memory_order_relaxed), false, r->window, ++r->probes_made, us,
                         hipSuccess});
    r->window = Delta();
    r->probed_upto = launched;
    return r->probes_made;
}

// An event behind the drain kernel of such a probe, once a flush has polled its words for kPollNs, and so in any case before the flush
// gives up: whoever comes upon the probe from then on can wait for it like for any other, and learns of a GPU that has failed.
static dmi_status_t event_behind(dmi_ring *r, uint64_t no)
{
    std::lock_guard<std::mutex> lk(r->pmu);
    for (Probe &p : r->probes) {
        if (p.no != no || p.ev) continue;
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (!capture_status(p.stream, &cs) || cs != hipStreamCaptureStatusNone) return DMI_OK;      // (it would end up in the graph)
        hipEvent_t ev = nullptr;
        p.failed = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (p.failed == hipSuccess && (p.failed = hipEventRecord(ev, p.stream)) != hipSuccess) (void)hipEventDestroy(ev);
        if (p.failed != hipSuccess) return fail(DMI_ERR_HIP, "event behind a flush's copy: %s", hipGetErrorString(p.failed));
        p.ev = ev;
    }
    return DMI_OK;
}

// Take note of finished probes: the slot of the newest launch they cover says where the
// device head stands.  With block=true waits for the oldest outstanding probe.
dmi_status_t advance_commits(dmi_ring *r, bool block)
{
    std::unique_lock<std::mutex> lk(r->pmu);
    const uint64_t oldest = r->probes.empty() ? 0u : r->probes.front().no;
    while (!r->probes.empty()) {
        Probe &p = r->probes.front();
        block = block && p.no == oldest;
        hipError_t e;
        if (p.failed != hipSuccess) {
            e = p.failed;
        } else if (p.note.groups && p.note.over()) {
            e = hipSuccess;
        } else if (p.ev) {
            e = block ? hipEventSynchronize(p.ev) : hipEventQuery(p.ev);
        } else if (block) {         // (another thread's flush polls it, and will put an event there)
            lk.unlock();
            std::this_thread::sleep_for(std::chrono::microseconds(10));
            lk.lock();
            continue;
        } else {
            e = hipErrorNotReady;
        }
        block = false;
        if (e == hipErrorNotReady) break;
        if (e != hipSuccess) return fail(DMI_ERR_HIP, "commit event: %s", hipGetErrorString(e));
        if (p.fetched) {
            const volatile CommitSlot &sl = r->hslots[(p.covers - 1u) % kCommitSlots];
            std::atomic_thread_fence(std::memory_order_acquire);
            if (sl.seq_plus1 != p.covers)
                return fail(DMI_ERR_CLOSED, "commit slot of launch %llu holds %llu",
                            (unsigned long long)(p.covers - 1u), (unsigned long long)sl.seq_plus1);
            r->snap[0] = sl.captured_records; r->snap[1] = sl.captured_rows; r->snap[2] = sl.captured_bytes;
            r->snap[3] = sl.dropped_records;  r->snap[4] = sl.dropped_rows;  r->snap[5] = sl.dropped_bytes;
            r->committed.store(sl.head, std::memory_order_release);
        } else {
            // state after the previous probe is exact, and so is what came since
            r->snap[0] += p.delta.records; r->snap[1] += p.delta.rows; r->snap[2] += p.delta.bytes;
            r->snap[3] += p.delta.drop_records; r->snap[4] += p.delta.drop_rows; r->snap[5] += p.delta.drop_bytes;
            r->committed.store(r->committed.load(std::memory_order_relaxed) + p.delta.bytes,
                               std::memory_order_release);
        }
        r->confirmed.store(p.covers, std::memory_order_release);
        r->confirmed_launches.store(p.launches, std::memory_order_release);
        r->probes_done.store(p.no, std::memory_order_release);
        if (p.ev) r->probe_pool.push_back(p.ev);
        r->probes.pop_front();
    }
    return DMI_OK;
}

uint64_t read_committed(const dmi_ring *r) { return r->committed.load(std::memory_order_acquire); }

// Up to where the device ring is complete: the head as the last probe has confirmed it or as a launch has noted it since.  Not by
// notes between dmi_step_begin and dmi_step_end: the captures of a replay belong to the drain, and to the counters, from the latter on.
// And never past what the host counts on as the head: the captures of a step that is destroyed before its end have noted more.
// Producer thread only.
static uint64_t read_complete(dmi_ring *r)
{
    if (r->step_open) return read_committed(r);
    const uint64_t noted = __atomic_load_n(r->hwords + kWordNote, __ATOMIC_ACQUIRE);
    return std::max(read_committed(r), std::min(noted, head_upper_bound(r)));
}

// The drained-up-to mark, where the kernels read it: one pinned word, written here and read by a
// lane of a running kernel across the host link at any time, so the store is an atomic one.
static void publish_tail(dmi_ring *r, uint64_t mark)
{
    __atomic_store_n(r->htail, mark, __ATOMIC_RELEASE);
}

// Retire finished copies (all of them at once: the drain stream is idle).  Caller holds r->mu.
dmi_status_t reap(dmi_ring *r)
{
    if (r->drain_done.load(std::memory_order_relaxed) == r->drain_issued) return DMI_OK;
    if (r->direct_probe) {      // on the producer's stream: the drain stream's being idle says nothing
        if (r->probes_done.load(std::memory_order_acquire) < r->direct_probe) return DMI_OK;
        r->direct_probe = 0;
        r->drain_done.store(r->drain_issued, std::memory_order_release);
        publish_tail(r, r->drain_issued);
        return DMI_OK;
    }
    if (r->copy_note.groups && !r->copy_note.over()) return DMI_OK;
    r->copy_note.groups = 0;
    if (r->copies) {
        hipError_t e = hipStreamQuery(r->drain_stream);
        if (e == hipErrorNotReady) return DMI_OK;
        if (e != hipSuccess) return fail(DMI_ERR_HIP, "drain stream: %s", hipGetErrorString(e));
        r->copies = false;
    }
    r->drain_done.store(r->drain_issued, std::memory_order_release);
    publish_tail(r, r->drain_issued);
    return DMI_OK;
}

// Workgroups of a drain kernel for n bytes.
static uint32_t drain_groups(uint64_t n)
{
    const uint64_t groups = (n / 16u + kThreads - 1u) / kThreads;
    return (uint32_t)(groups < kDrainGroups ? groups : kDrainGroups);
}

// Copy stream bytes [from, from + n) on the drain stream.  Caller holds r->mu.
static dmi_status_t copy_span(dmi_ring *r, uint64_t from, uint64_t n)
{
    r->copies = true;
    if (r->cfg.flags & DMI_DRAIN_KERNEL) {
        HIP_TRY(launch_drain_kernel(r->dev_ring, r->dev_cap, r->host_ring_dev, r->host_cap, from, n, drain_groups(n), nullptr, 0u,
                                    r->drain_stream));
        return DMI_OK;
    }
    while (n) {
        const uint64_t s = from % r->dev_cap, d = from % r->host_cap;
        uint64_t len = n;
        if (len > r->dev_cap - s) len = r->dev_cap - s;
        if (len > r->host_cap - d) len = r->host_cap - d;
        HIP_TRY(hipMemcpyAsync(r->host_ring + d, r->dev_ring + s, len, hipMemcpyDeviceToHost, r->drain_stream));
        from += len;
        n -= len;
    }
    return DMI_OK;
}

// The same by a drain kernel that says itself when it is over, on a stream of its own (nothing is in front of it there and it
// waits for nothing).  One at a time.
static dmi_status_t copy_span_noted(dmi_ring *r, uint64_t from, uint64_t n)
{
    const DrainNote note = {r->hwords + kWordsDrain, drain_groups(n), ++r->drain_tick};
    HIP_TRY(launch_drain_kernel(r->dev_ring, r->dev_cap, r->host_ring_dev, r->host_cap, from, n, note.groups,
                                r->hwords_dev + kWordsDrain, note.tick, r->ctl_stream));
    r->copy_note = note;
    return DMI_OK;
}

// Has the producer's stream nothing on it?  (Under capture, or if the runtime will not say: taken for no; a query would end the capture.
// Cheap where an event is the last thing on the stream, as it is when the captures are known to be over and nothing is behind them; behind
// a kernel the runtime first puts a marker there to ask for: 28 us for a flush that asked behind its drain kernel.)
static bool producer_is_idle(const dmi_ring *r)
{
    hipStream_t us = (hipStream_t)r->last_stream.load(std::memory_order_acquire);
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (r->quiet.load(std::memory_order_acquire) || !capture_status(us, &cs) || cs != hipStreamCaptureStatusNone) return false;
    if (hipStreamQuery(us) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Issue copies for what is complete and fits the host ring.  Caller holds r->mu.  Complete is what a probe has confirmed, for
// `flush` also what a launch has noted: a flush by the producer's own thread, which polls and knows how much is still to come (other
// drains would copy whatever a note happens to say, and every copy costs the link some 8 us).  While captures are still running, one copy
// at a time of at least flush->least bytes, by the copy engine: a drain kernel beside them has them wait behind its stores across the link (32
// captures of 64 x 4096 took ten times as long as long as one ran).  Behind the captures, if the producer's stream has come to its end
// there, a drain kernel, which starts 5 us sooner than the copy engine (from the captures' end to the host's knowing of the
// copy's: 4 KB 7.7 / 12.3 us, 2 MB 45.5 / 46.5, 4.2 MB 83 / 88, 16.8 MB 311 / 311), also beside a copy that is under way.  Where the caller's
// next kernels run there, its workgroups wait for places among theirs: 4.2 MB with 2.4 ms of matrix
// products behind the captures are there after 305 us by the copy engine, and by a drain kernel after 1040.  And what is
// left of a span that went in several copies stays with the copy engine, which has just been at it (64 MiB and 2.4 MB behind them: 1299 us, with
// a drain kernel for those 1306).
dmi_status_t drain_issue_locked(dmi_ring *r, uint64_t *moved, bool *host_full, const ChunkRule *flush)
{
    if (moved) *moved = 0;
    if (host_full) *host_full = false;
    dmi_status_t st = reap(r);
    if (st != DMI_OK) return st;
    if (r->direct_probe) return DMI_OK;
    uint64_t committed, committed_records;
    {   // the head and the record count that belong to it
        std::lock_guard<std::mutex> pk(r->pmu);
        committed = read_committed(r);
        committed_records = r->snap[0];
    }
    // (a flush by notes that has given up may have gone further than an event has confirmed)
    const uint64_t complete = std::max(flush ? read_complete(r) : committed, r->drain_issued);
    atomic_max(r->dev_high, complete - r->drain_done.load(std::memory_order_relaxed));
    const uint64_t avail = complete - r->drain_issued;
    if (flush && flush->more && (r->copies || avail < flush->least)) return DMI_OK;
    if (flush && r->copy_note.groups) return DMI_OK;
    const uint64_t host_free = r->host_cap - (r->drain_issued - r->released);
    uint64_t n = avail < host_free ? avail : host_free;
    if (host_full) *host_full = avail > 0 && host_free == 0;
    // bounded batches: the device tail (what drop-newest decides on) moves once per batch
    const uint64_t batch = (r->dev_cap / 8u > (64u << 20) ? r->dev_cap / 8u : (64u << 20)) & ~63ull;
    if (n > batch) n = batch;
    if (n > 0) {
        const uint64_t from = r->drain_issued;
        if (flush && !flush->more && !flush->engine && n <= kChunkKernelBytes && producer_is_idle(r)) {
            if ((st = copy_span_noted(r, from, n)) != DMI_OK) return st;
        } else {
            if ((st = copy_span(r, from, n)) != DMI_OK) return st;
        }
        r->drain_issued = from + n;
        if (r->drain_issued == committed) r->drain_issued_records = committed_records;
        r->drained_bytes += n;
        r->drain_batches += 1;
        atomic_max(r->host_high, r->drain_issued - r->released);
        if (moved) *moved = n;
    }
    return DMI_OK;
}

// Issue the copies and, if asked, wait for them.  The ring's lock is held only while the
// bookkeeping is touched, never across the wait: the consumer polls and releases, and the
// producer asks for room, while a copy is in flight.
dmi_status_t drain(dmi_ring *r, bool wait, uint64_t *moved, bool *host_full, const ChunkRule *flush)
{
    uint64_t mark;
    bool noted;
    {
        std::lock_guard<std::mutex> lk(r->mu);
        dmi_status_t st = drain_issue_locked(r, moved, host_full, flush);
        if (st != DMI_OK) return st;
        mark = r->drain_issued;
        if (!wait || r->direct_probe || r->drain_done.load(std::memory_order_relaxed) == mark) return DMI_OK;
        if (flush && (flush->more || (flush->poll && r->copy_note.groups))) return DMI_OK;
        noted = r->copy_note.groups != 0;
    }
    // everything issued up to `mark` was on these streams before this call
    hipError_t e = hipStreamSynchronize(r->drain_stream);
    if (e == hipSuccess && noted) e = hipStreamSynchronize(r->ctl_stream);
    if (e != hipSuccess) return fail(DMI_ERR_HIP, "drain stream: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lk(r->mu);
    if (r->drain_done.load(std::memory_order_relaxed) < mark) {
        r->drain_done.store(mark, std::memory_order_release);
        publish_tail(r, mark);  // the span may be reused only now that its copies have run
        if (mark == r->drain_issued) { r->copies = false; r->copy_note.groups = 0; }
    }
    return DMI_OK;
}

// Between two looks at something that the GPU is about to finish.  In the producer's own thread at
// first only the processor is offered to others (a sleep of 10 us takes some 60 here, longer than most of
// what a flush waits for).  Any other thread sleeps: every look takes a lock that each observe takes too.  A
// second thread that flushed back to back without sleeping took a producer's observe of 64 x 4096 from 3.2 us
// (median; nine in ten below 5.4) to 4.8 (16.1).
static void pause_since(const dmi_ring *r, uint64_t t0)
{
    if (r->producer.load(std::memory_order_relaxed) == this_thread() && now_ns() - t0 < 500000u) std::this_thread::yield();
    else std::this_thread::sleep_for(std::chrono::microseconds(10));
}

// A flush whose bytes the host can tell in advance: the drain kernel moves them on the producer's
// own stream, right behind the captures, and says itself when it is over.  Otherwise the host waits
// for the captures' event, only then starts a copy, and waits for that.  *probe: the probe that says when it is over; 0 if this was not done.
// Measured from a capture's launch to the end of the wait, drain kernel against event and copy engine:
// 10.0 / 23.4 us for 4 KB, 21.4 / 31.5 for 0.6 MB, 47.5 / 57.5 for 2 MB, 85 / 99.5 for 4.2 MB.  Not above 6 MiB, where the kernel's 64
// workgroups would be on the GPU for more than 100 us to save a tenth of that.
// Left to the copy engine: a flush by any other thread than the producer's, which goes on launching its
// model's kernels meanwhile and would find the copy in front of them on their stream; a ring whose creator
// asked for the copy engine by name; a ring with a drain thread (it follows the commits and issues copies by
// itself at any time); sizes only the device knows (drops or keep vectors decided there); a span the host ring
// has no room for as a whole, or behind copies still under way.  And, whole, a span part of which has a
// probe behind it already (every sixteenth launch puts one there, and the end of a replayed step) or is known to
// be captured: those bytes need not wait for what the caller has put on the stream since, which the copy behind
// it all would.  A launch without a probe gets one now, behind all that, so there the copy waits for nothing more.
static dmi_status_t flush_behind_captures(dmi_ring *r, uint64_t *moved, uint64_t *probe)
{
    *probe = 0;
    if (r->cfg.flags & (DMI_BG_THREAD | DMI_DRAIN_COPY_ENGINE)) return DMI_OK;
    if (r->producer.load(std::memory_order_relaxed) != this_thread()) return DMI_OK;
    std::lock_guard<std::mutex> lk(r->mu);
    dmi_status_t st = reap(r);
    if (st != DMI_OK) return st;
    if (r->direct_probe || r->drain_done.load(std::memory_order_relaxed) != r->drain_issued) return DMI_OK;
    uint64_t target, records;
    {
        std::lock_guard<std::mutex> pk(r->pmu);
        if (!r->window_exact || !r->probes.empty() || r->next_seq.load(std::memory_order_acquire) <= r->probed_upto ||
            read_committed(r) > r->drain_issued)
            return DMI_OK;
        target = read_committed(r) + r->window.bytes;
        records = r->snap[0] + r->window.records;
    }
    const uint64_t from = r->drain_issued, n = target - from;
    if (n == 0 || n > kFlushKernelBytes || n > r->host_cap - (from - r->released)) return DMI_OK;
    // what notes say, or will still say while later captures run, need not wait for those
    const uint64_t complete = read_complete(r);
    if (complete >= from + kLeastChunk || target >= r->unnoted_bytes + complete + kWorthNotes) return DMI_OK;
    // Not while the stream is being captured: the copy would end up in the graph.
    hipStream_t us = (hipStream_t)r->last_stream.load(std::memory_order_acquire);
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (r->quiet.load(std::memory_order_acquire) || !capture_status(us, &cs) || cs != hipStreamCaptureStatusNone)
        return DMI_OK;
    atomic_max(r->dev_high, n);
    const DrainNote note = {r->hwords + kWordsBehind, drain_groups(n), ++r->drain_tick};
    HIP_TRY(launch_drain_kernel(r->dev_ring, r->dev_cap, r->host_ring_dev, r->host_cap, from, n, note.groups,
                                r->hwords_dev + kWordsBehind, note.tick, us));
    // (a probe of its own, even if another thread's drain has just put one there: that one may be in front of the
    // copy; this thread is the producer, whose count of launches starts again behind it)
    const uint64_t no = probe_by_drain(r, note, us);
    r->unprobed_launches = 0;
    r->unprobed_bytes = 0;
    r->direct_probe = no;
    r->drain_issued = target;
    r->drain_issued_records = records;
    r->drained_bytes += n;
    r->drain_batches += 1;
    atomic_max(r->host_high, target - r->released);
    *moved = n;
    *probe = no;
    return DMI_OK;
}

// A drain that waits does so for a flush's span on the producer's stream too, as it does for copies
// issued earlier (another thread's flush, or one that gave up waiting): at most block_timeout_ms, because
// the producer's stream may be busy with the caller's own work.
static dmi_status_t wait_for_direct(dmi_ring *r)
{
    const uint64_t t0 = now_ns();
    for (;;) {
        {
            std::lock_guard<std::mutex> lk(r->mu);
            dmi_status_t st = reap(r);
            if (st != DMI_OK || !r->direct_probe) return st;
        }
        if (now_ns() - t0 > (uint64_t)r->block_timeout_ms * 1000000ull)
            return fail(DMI_ERR_AGAIN, "the copy of an earlier flush did not finish within %u ms", r->block_timeout_ms);
        pause_since(r, t0);
        dmi_status_t st = advance_commits(r, false);
        if (st != DMI_OK) return st;
    }
}

// Pop launches known to have finished; returns an upper bound of the device head once
// everything launched so far has run.  Producer thread only.
uint64_t head_upper_bound(dmi_ring *r)
{
    const uint64_t done = r->confirmed.load(std::memory_order_acquire);
    const uint64_t committed = r->committed.load(std::memory_order_acquire);
    while (!r->inflight.empty() && r->inflight.front().first < done) {
        r->inflight_sum -= r->inflight.front().second;
        r->inflight.pop_front();
    }
    return committed + r->inflight_sum;
}

// Completeness policy: wait on the host until a record of `ub` bytes is sure to fit
// (the paper's flush before the forward step, section 4.4).  Never a device-side wait.
dmi_status_t wait_for_room(dmi_ring *r, uint64_t ub)
{
    uint64_t t0 = 0;
    dmi_status_t st;
    for (;;) {
        // what the drain side has confirmed so far is enough to decide in the common case
        // (an older view only makes the bound more cautious)
        uint64_t head_ub = head_upper_bound(r);
        uint64_t tail = r->drain_done.load(std::memory_order_acquire);
        if (head_ub - tail + ub <= r->dev_cap) break;
        if ((st = advance_commits(r, false)) != DMI_OK) return st;
        head_ub = head_upper_bound(r);
        tail = r->drain_done.load(std::memory_order_acquire);
        if (head_ub - tail + ub <= r->dev_cap) break;
        if (!t0) t0 = now_ns();
        uint64_t moved = 0;
        if ((st = drain(r, true, &moved)) != DMI_OK) return st;
        if (moved) continue;
        st = record_probe(r);       // make sure the launches we wait for will report
        if (st != DMI_OK) return st;
        if (now_ns() - t0 > (uint64_t)r->block_timeout_ms * 1000000ull) {
            r->block_wait_ns += now_ns() - t0;
            return fail(DMI_ERR_AGAIN, "no room in the device ring after %u ms (host ring full or "
                                       "observes not finishing)", r->block_timeout_ms);
        }
        std::this_thread::sleep_for(std::chrono::microseconds(10));
    }
    if (t0) r->block_wait_ns += now_ns() - t0;
    return DMI_OK;
}

// A launch's commit slot is reused kCommitSlots launches later: keep fewer than that
// unconfirmed before issuing `n` more.
dmi_status_t commit_slot_room(dmi_ring *r, uint32_t n)
{
    while (r->next_seq.load(std::memory_order_relaxed) + n - r->confirmed.load(std::memory_order_acquire) >=
           kCommitSlots) {
        dmi_status_t st = record_probe(r);
        if (st == DMI_OK) st = advance_commits(r, true);
        if (st != DMI_OK) return st;
    }
    return DMI_OK;
}

// Request table as the kernels read it: n x {req_id, tok_start, tok_step, tok_count}, then
// n x first source row of the request (dense; callers have checked that it fits 32 bits)
// or its row of the block table (paged); with row_map, then the source row of every listed
// row in output order (for the decode-shaped kernel when requests list several rows).
void selection_words(const dmi_req_sel_t *reqs, uint32_t n, bool paged, bool row_map, std::vector<uint32_t> &words)
{
    words.resize((size_t)n * 5u);
    for (uint32_t i = 0; i < n; i++) {
        const dmi_req_sel_t &q = reqs[i];
        words[4u * i + 0] = q.req_id;
        words[4u * i + 1] = q.tok_start;
        words[4u * i + 2] = q.tok_step;
        words[4u * i + 3] = q.tok_count;
        words[4u * n + i] = paged ? q.row_base : q.row_base + q.tok_start;
    }
    if (row_map)
        for (uint32_t i = 0; i < n; i++)
            for (uint32_t j = 0; j < reqs[i].tok_count; j++)
                words.push_back(reqs[i].row_base + reqs[i].tok_start + j * reqs[i].tok_step);
}

// Put the request table where the kernel can read it from L2: a slab of slots in
// device memory, refilled only when the selection differs from recent ones (all
// hook points of a step share their selection).
dmi_status_t stage_selection(dmi_ring *r, const dmi_selection_t *sel, bool paged, bool row_map, hipStream_t s,
                             uint32_t *slot_out)
{
    std::vector<uint32_t> &words = r->sel_scratch;
    selection_words(sel->reqs, sel->n_reqs, paged, row_map, words);
    for (auto &c : r->cache) {
        if (!c.valid || c.stream != s || c.paged != paged || c.words.size() != words.size()) continue;
        if (words.empty() || memcmp(c.words.data(), words.data(), words.size() * 4u) == 0) {
            *slot_out = c.slot;
            return DMI_OK;
        }
    }
    const uint32_t slot = r->next_slab++ % kSlabSlots;
    for (auto &c : r->cache) if (c.valid && c.slot == slot) c.valid = false;
    if (!words.empty())
        HIP_TRY(launch_upload(r->slab + (size_t)slot * r->slab_slot_words, words.data(), (uint32_t)words.size(), s));
    SelCache &c = r->cache[r->cache_rr++ % kSelCache];
    c.valid = true; c.paged = paged; c.stream = s; c.slot = slot; c.words = words;
    *slot_out = slot;
    return DMI_OK;
}

// Fill every kernel argument that depends only on the tensor, the selection's shape and the
// transform.  Left to the caller: request table location, sequence number, step id, commit
// slot, tail floor, policy, chain parity.
// Workgroups per tensor (gridDim.x) of the general kernel for a launch of `nb` tensors.
// Work items per launch path, and a grid that gives every workgroup the same number of them:
// with a fixed grid of "as many as fit" the last round is run by a fraction of the
// workgroups while the rest idle (up to half the launch for 1 < items/grid < 2).
// kResident is five workgroups per compute unit: the kernels hold from four (summaries of short rows off the 16-byte grid:
// up to 118 vector registers) to eight (rows dealt flat: 45 to 51); they are all planned for five.  In a batch (gridDim.y = nb) each workgroup stays with one tensor.
// `of`: the tensors that this launch and its neighbours read one after the other, if those are more (what is left of them in the
// memory-side cache is a matter of them all).
uint32_t plan_grid(CaptureArgs &a, uint32_t nb, uint32_t of)
{
    if (of < nb) of = nb;
    constexpr uint64_t kResident = 5u * 256u;
    const uint64_t listed = a.listed_rows, upr = a.units_per_row;
    // Decode-like selections (one row per request, no keep vector, dense) need no scan and no
    // search: a workgroup per item, each gone after one round trip, keeps more loads in flight
    // than the resident few looping over many items.
    const bool flat = a.simple && !a.paged;
    // capture_rows_kernel scans the table with a request per lane
    const bool finds_rows_itself = !a.paged && (a.simple || (a.n_reqs >= 1u && a.n_reqs <= 64u));
    // Rows that a record is expected to have.  With a keep vector that the host does not know: half of the listed ones, but
    // never fewer workgroups than fill the GPU while there are rows for them.  A workgroup that finds itself behind the last kept
    // row has spent a microsecond and a place on a compute unit to learn that; on a GPU that is not full that costs nothing, and
    // a row that waits for another one costs a trip to memory.  (Planned for the kept rows / half / all, us: 16.4 k listed rows of
    // 1024 units fp32, statistics, 14 % kept 9.5 / 11.3 / 14.1, 52 % 23.1 / 23.1 / 24.6, 100 % 39.1 / 40.4 / 39.1; stored 14.3 / 15.3 / 18.3,
    // 43.0 / 43.0 / 45.3, 80.0 / 81.2 / 80.0; 1 k listed rows of 1024, 100 % 4.4 / 5.7 / 4.4; 4.1 k of 512, statistics, 45 % - / 5.6 / 4.3,
    // 100 % 6.1 / 9.0 / 6.1; 55 rows of 1024, 100 % 4.1 / 4.6 / 4.1.)
    constexpr uint64_t kFull = 8u * 256u;       // workgroups
    const bool guess = a.keep_mask && !a.rows_known;
    const uint64_t expected = a.rows_known ? a.kept_rows : guess ? (listed + 1u) / 2u : listed;
    auto planned = [&](auto groups_for) -> uint64_t {       // workgroups for as many rows
        const uint64_t n = groups_for(expected), full = (kFull + nb - 1u) / nb;
        return guess && n < full ? std::min(groups_for(listed), full) : n;
    };
    // A launch reads past the memory-side cache (non-temporal loads) if it reads more than that holds, or at least half as much out of a
    // stretch of rows that is larger: such a stretch has just gone through the cache and left its end there, in lines that have to be
    // written back for every row that is brought in, and the next kernel that goes through it finds next to nothing of it either way.
    // (Through / past the cache, us, rows written by the kernel before; behind the + a sum over the whole stretch behind the launch.  To fp8,
    // 265 MB of 1063 113 + 301 / 73 + 314, of 531 109 + 163 / 72 + 174, 132 of 1061 59 + 309 / 38 + 319, of 530 51 + 171 / 39 + 177, all of
    // 300 85 + 95 / 67 + 94; raw 265 of 1063 139 + 302 / 94 + 316; statistics 85 + 300 / 44 + 315.  On cold rows 74 / 71, 72 / 70, 40 / 39, 40 / 39,
    // 80 / 77.)  Of a smaller part enough may have stayed in the cache (75 MB of 303, cold 25 + 95 / 24 + 99, written 22 + 106 / 20 + 111), and a
    // stretch that it holds is found there, and left there, only through it (265 MB, all read: 62 + 74 / 59 + 88, cold 71 + 68 / 70 + 88; 132
    // of 265 33 + 71 / 32 + 86; statistics 22 + 73 / 26 + 86).
    constexpr uint64_t kMemorySideCache = 256ull << 20;
    const uint64_t row_bytes = (uint64_t)a.row_elems * dtype_size(a.src_dtype), source_bytes = expected * of * row_bytes;
    const uint64_t stretch_bytes = a.stretch_rows ? of * ((a.stretch_rows - 1u) * (uint64_t)a.row_stride_b + row_bytes) : 0u;
    const bool past_the_cache = source_bytes > kMemorySideCache ||
                                (stretch_bytes > kMemorySideCache && source_bytes >= kMemorySideCache / 2u);
    // A batch's tensors have been kept for this launch and nothing reads them behind it: from half of the cache on.  (Through / past the
    // cache, cold and just written: statistics alone 134 MB 25.1 / 24.4 and 21.3 / 20.9, 200 MB 34.9 / 34.1 and 29.7 / 29.0; 256 x 8192 raw, 24 tensors
    // 37.0 / 37.0 and 31.5 / 31.5, 32 49.2 / 47.2 and 40.8 / 40.8, 40 60.5 / 57.7 and 50.4 / 49.9, 48 72.0 / 67.9 and 59.9 / 59.5; with statistics 48
    // 71.1 / 69.6 and 62.9 / 63.0; to fp8 56.9 / 56.4 and 49.2 / 49.3; 3 x 9.2 k x 4096 raw 80.6 / 79.4 and 66.7 / 67.5.)
    const bool batch_past_the_cache = of > 1u && source_bytes >= kMemorySideCache / 2u;
    a.step_per_wave = a.read_once = a.wave_rows = 0;
    // A launch of several tensors works through them one after the other (the y index of a workgroup
    // is the slow one), and does best with short-lived workgroups of about four items each: the
    // hardware then hands out the work as workgroups retire, which evens out how unequally the
    // workgroups are served (the five that share a compute unit oldest first: with equal shares the
    // youngest ends 1.4 times as late as the oldest; and compute units differ by +-8 %), while
    // workgroups that stay for a whole tensor all have to end before the next tensor's can start,
    // and a resident set shared among the tensors leaves every tensor's tail to a few workgroups.
    constexpr uint64_t kItemsPerGroupInBatch = 4u;
    auto balanced = [nb, flat](uint64_t items, uint64_t most) -> uint64_t {
        if (flat || items * nb <= kResident) return items;
        uint64_t rounds = (items * nb + kResident - 1u) / kResident;
        if (nb > 1u && rounds > most) rounds = most;
        return (items + rounds - 1u) / rounds;
    };
    // Rows stored without summaries, of at least kLongRowUnits units: a wavefront per 256 units of one (capture_rows_kernel).  It
    // takes its time also where its step is short: from 12 k steps on rows go there if those are long enough, else they are dealt flat.
    // (rows kernel / dealt flat, us; one row per request: 32.8 k rows of 64 units raw 15.5 / 14.9, of 80 16.5 / 16.9; fp16 of 72
    // 18.7 / 16.7, of 80 18.8 / 18.0, of 96 21.5 / 22.8; fp8 of 64 18.5 / 14.0, of 96 21.2 / 19.3, of 112 21.6 / 21.9; 24 k to fp8 of 104 15.4 / 15.5;
    // ragged: 40 k of 64 raw 21.1 / 17.3, of 72 20.9 / 19.2, of 80 21.1 / 21.8; fp16 of 96 30.1 / 27.6, 24 k of 104 17.1 / 18.3; fp8 of 64
    // 23.8 / 14.9, of 128 30.1 / 28.1, of 136 32.3 / 32.5, of 257 59.1 / 51.5.  Smaller launches: 8 k of 64 raw 7.4 / 7.4, fp8 8.0 / 9.2,
    // 1.5 k 4.2 / 6.1 and 4.9 / 6.8; 12 k of 64 ragged raw 9.1 / 8.0, 10 k 8.1 / 7.9.)
    const uint64_t steps_per_row = (upr + 255u) / 256u;
    const uint64_t least = a.out_dtype == a.src_dtype ? (a.simple ? 72u : 80u) : a.out_dtype == DMI_DTYPE_FP8_E4M3FN ? (a.simple ? 104u : 136u)
                                                                                                                      : (a.simple ? 80u : 104u);
    const bool rows_of_steps = finds_rows_itself && upr >= kLongRowUnits &&
                               (upr >= least * steps_per_row || expected * nb * steps_per_row < 12000u);
    uint64_t groups;
    // Rows of 129 to 256 units have a wavefront's lanes to themselves either way; in capture_rows_kernel they come without the
    // general kernel's prologue (12.8 k rows of 256 units, statistics 13.8 -> 10.9 us, stored too 20.9 -> 18.4; 3 k of 192
    // 6.3 -> 4.1; off the 16-byte grid 19.0 -> 13.2; 80 x 256 rows of 256 in one launch 27.1 -> 18.4).  Not statistics alone of
    // very many of the shortest of them (40 k rows of 130 units: 20.4 and 21.9).
    const bool own_wavefront = finds_rows_itself && a.row_lanes == 64u && (upr >= 192u || a.out_dtype || listed * nb < 32768u);
    if (a.summary_mask && a.row_lanes <= 64u && !own_wavefront) {
        const uint64_t rows = 4u * (64u / a.row_lanes);             // what a workgroup takes in one step
        // (statistics alone, 8 caches x 72.7 k rows of 32 units: 66 us, past the cache 60; of 128 units 118, 104, and with eight
        // items per workgroup 101)
        a.read_once = !a.out_dtype && past_the_cache;
        groups = balanced((listed + rows - 1u) / rows, a.out_dtype ? kItemsPerGroupInBatch : 8u);
    } else if (a.summary_mask && finds_rows_itself) {
        // capture_rows_kernel: a wavefront per row while a launch has rows enough to fill the GPU that way and they are
        // short enough for one wavefront's trips, else a workgroup per row, a quarter of it to each wavefront.
        // (workgroup / wavefront per row / the general kernel, norm and largest magnitude, us; ragged, 16 to 32 requests:)
        //   statistics alone: 12.8 k rows of 264 units 21.9 / 12.6 / 15.1, 9.3 k rows of 512 17.2 / 13.9 / 16.4, of 513 off the
        //   16-byte grid 22.6 / 17.4 / 24.0, of 768 24.1 / 22.9 / 24.4, of 1024 27.6 / 32.7 / 32.4, of 2048 54.1 / 67.8 / 60.5,
        //   200 of 6283 9.2 / 25.4 / 13.3
        //   rows stored too: 9.3 k of 384 21.4 / 20.5 / 20.7, of 512 26.1 / 25.4 / 25.5, of 768 40.4 / 47.4 / 46.4, of 1024
        //   53.2 / 66.8 / 63.8, of 2048 113.8 / 153.6 / 129.4
        //   batches, one row per request: 80 x 256 rows of 512 39.5 / 30.9 / 33.1, of 1024 57.4 / 62.5 / 62.6 (rows stored too 120 / 138
        //   / 116, and 115 past the cache)
        a.step_per_wave = 1;
        a.wave_rows = upr <= 256u || (upr <= 640u && (guess ? listed : expected) * nb >= 2048u);
        a.read_once = past_the_cache || batch_past_the_cache;
        groups = planned([&](uint64_t rows) { return a.wave_rows ? (rows + 3u) / 4u : rows; });
    } else if (a.summary_mask) {
        // Rows of more than 256 units of paged caches, or of more than 64 ragged requests: a workgroup per row, or, where a
        // launch has rows enough, a wavefront per row.
        // (workgroup / wavefront per row, norm and largest magnitude, us:)
        //   rows of 288 units, 1.5 k rows 7.5 / 7.5, 3 k 10.0 / 7.4, 6 k 16.6 / 9.9; of 512: 24 k 57.3 / 40.0
        //   of 640 units, 6 k rows 17.3 / 14.4; 40 x 256 rows of 768, statistics alone 34.7 / 27.7, with the rows 45 / 49
        //   of 1024 units, 12 k rows 38.5 / 42.2, 18 k 56.4 / 59.3, 24 k 72.5 / 76.1 (of 800: 36.1 / 32.4 and
        //   63.7 / 62.4); of 1792 units, 12 k rows 66.6 / 69.4
        // With statistics alone a wavefront takes two rows from 4096 rows on (80 x 256 rows of 512 units: 37.2 with
        // one, 34.8 with two; 3 k rows 8.7 and 9.0), where the rows are stored too, one (61 and 64 us).
        const uint64_t rows = listed * nb;
        const bool alone = a.out_dtype == 0u;
        a.wave_rows = rows >= 2048u && (upr <= 512u || (alone && upr <= 768u));
        const uint64_t per_wave = alone && rows >= 4096u ? 2u : 1u;
        groups = a.wave_rows ? (listed + 4u * per_wave - 1u) / (4u * per_wave) : balanced(listed, kItemsPerGroupInBatch);
    } else if (a.out_dtype && rows_of_steps) {
        a.step_per_wave = 1;
        a.read_once = past_the_cache || batch_past_the_cache;
        groups = planned([&](uint64_t rows) { return (rows * steps_per_row + 3u) / 4u; });
    } else {
        // Short rows: slices of 256 units; a workgroup takes 4 per round once there are enough.  In a batch of up to nine rounds
        // the resident set shared evenly, then two items per workgroup, from twenty on four as above: eight workgroups of this path
        // share a compute unit, and with four items each the middling sizes left the last of them alone.  (Four / two / shared, cold
        // and just written, us; paged, rows of 32 units raw: 6.5 rounds 62.5 / 56.8 / 57.4 and 77.0 / 70.6 / 65.3, 7.8 68.6 / 68.5 / 67.1 and
        // 83.2 / 83.8 / 76.7, 9.0 76.3 / 76.2 / 79.2 and 95.1 / 94.2 / 92.9, 10.3 91.2 / 87.5 / 87.0 and 110.6 / 106.0 / 101.4, 11.6 99.6 / 94.8 and
        // 120.7 / 115.0, 23 183.4 / 181.7 / 192.1 and 206.1 / 202.6 / 215.7, 94 594 / 601 and 646 / 667; to fp8 6.5 52.8 / 46.9 / 48.0, 11.6 80.3 / 76.9, 23
        // 143.8 / 145.1 / 154.7, 94 430 / 446; 12 x 5.1 k ragged rows of 512 units to fp8, 24 rounds 142.8 / 149.5.)
        const uint64_t slices = (listed * upr + kThreads - 1u) / kThreads, items = (slices + 3u) / 4u;
        const uint64_t most = items * nb <= 9u * kResident ? 9u : items * nb <= 20u * kResident ? 2u : kItemsPerGroupInBatch;
        groups = slices * nb <= kResident ? slices : balanced(items, most);
    }
    return groups < 1u ? 1u : groups > kMaxGrid ? kMaxGrid : (uint32_t)groups;
}

} }  // namespace dmi::host
namespace dmi {
// Which launches the decode-shaped kernel can take (see capture_decode_kernel).
bool decode_kernel_applies(const CaptureArgs &a, bool vec16)
{
    // one row per request (with a keep vector: up to 1024 requests), or, without a keep vector, any
    // selection of at most 1024 rows (the host then lists the source row of every output row)
    const bool shape = a.simple || (a.one_row_each && a.keep_mask && a.n_reqs <= 1024u) ||
                       (!a.keep_mask && a.listed_rows >= 1u && a.listed_rows <= kDecodeMaxListed);
    // 16-bit sources: bf16 with any supported output, fp16 as it is (or summaries only)
    const bool types = a.src_dtype == 1u || (a.src_dtype == 2u && (a.out_dtype == 2u || a.out_dtype == 0u));
    return shape && !a.paged && vec16 && types && a.units_per_row <= 4u * kThreads && a.n_reqs >= 1u;
}
}  // namespace dmi
namespace dmi { namespace host {

// Which kernel a launch of `nb` decode-shaped tensors takes.  The decode-shaped kernel is the
// quickest way through a small launch, where every dependent trip to memory counts; from
// some eight thousand rows on capture_rows_kernel's one-step wavefronts are as quick or quicker
// (measured on 256 x 8192 bf16 tensors: 13.3 against 15.2 us for 8 tensors, 44 us either way for
// 32, 116 against 113 us for 80).  The caller has set a.drop_newest and a.step.
bool batch_takes_decode_kernel(const CaptureArgs &a, uint32_t nb)
{
    if (nb == 1u) return true;
    // the decode-shaped kernel loads its row before it knows whether the record is dropped: fine for
    // one record, wasted reads for the dropped part of a batch under best effort (a replayable
    // step's policy is not known when it is captured)
    if (a.drop_newest || a.step) return false;
    return (uint64_t)nb * (a.listed_rows + 1u) <= 8192u;
}

// Element alignment of every source of a batch, and whether all of them allow 16-byte moves.
dmi_status_t check_batch_sources(uint32_t n, const void *const *data, uint32_t es, bool *all16)
{
    *all16 = true;
    for (uint32_t i = 0; i < n; i++) {
        if (!data[i]) return fail(DMI_ERR_INVALID_ARG, "data[%u] is NULL", i);
        if ((uintptr_t)data[i] % es) return fail(DMI_ERR_INVALID_ARG, "data[%u] is not element aligned", i);
        if ((uintptr_t)data[i] % 16u) *all16 = false;
    }
    return DMI_OK;
}

PlanEnv plan_env(const dmi_ring *r) { return PlanEnv{r->dev_ring, r->dev_cap, r->host_cap, r->dctrl, r->cfg.rank_tag, r}; }

dmi_status_t plan_capture(const PlanEnv &env, uint32_t point_id, const dmi_selection_t *sel, const dmi_transform_t *xf,
                          const Geometry &geo, CaptureArgs &a, Plan &pl, bool fixed_row_count_ok)
{
    const dmi_ring *r = env.masks;
    const uint32_t es_in = dtype_size(geo.src_dtype);
    uint64_t listed = 0, first = UINT64_MAX, end = 0;
    for (uint32_t i = 0; i < sel->n_reqs; i++) {
        const dmi_req_sel_t &q = sel->reqs[i];
        listed += q.tok_count;
        if (!q.tok_count) continue;
        const uint64_t at = (uint64_t)q.row_base + q.tok_start;
        first = std::min(first, at);
        end = std::max(end, at + (uint64_t)(q.tok_count - 1u) * q.tok_step + 1u);
    }
    a.stretch_rows = a.paged || sel->row_index_dev || end <= first ? 0u : end - first;     // (rows of a table or an index: unknown)
    // 16-byte units wherever a row (a head's part of a paged row) has 16 bytes, on a 16-byte grid or not;
    // shorter rows that are not on one go element by element.  64 rows x 50257 bf16: 12.0 us by elements, 4.9 in units; 9.3 k x 4099 to fp8: 133 and 34 us.
    a.loose = !geo.vec16 && geo.seg_elems >= 16u / es_in;
    const uint32_t unit_elems = geo.vec16 || a.loose ? 16u / es_in : 1u;
    a.seg_elems = geo.seg_elems;
    a.seg_units = (geo.seg_elems + unit_elems - 1u) / unit_elems;
    const uint64_t upr = (uint64_t)geo.n_seg * a.seg_units;
    a.limit_units = geo.vec16 ? (uint32_t)upr : geo.row_elems;
    if (listed > 0xFFFFFFFFull || listed * a.limit_units > 0xFFFFFFFFull)
        return fail(DMI_ERR_TOO_LARGE, "selection of %llu rows x %llu units exceeds one record",
                    (unsigned long long)listed, (unsigned long long)a.limit_units);
    const uint64_t ub = dmi_record_bytes(sel->n_reqs, listed, geo.row_elems, xf->out_dtype, xf->summary_mask);
    if (ub > env.cap)
        return fail(DMI_ERR_TOO_LARGE, "record of %llu bytes exceeds the device ring (%llu)",
                    (unsigned long long)ub, (unsigned long long)env.cap);
    if (env.host_cap && ub > env.host_cap)      // such a record could be drained but never polled whole
        return fail(DMI_ERR_TOO_LARGE, "record of %llu bytes exceeds the host ring (%llu)",
                    (unsigned long long)ub, (unsigned long long)env.host_cap);
    pl.listed = listed;
    pl.ub = ub;
    pl.rows_known = listed;
    pl.size_known = sel->keep_mask_dev == nullptr;
    if (fixed_row_count_ok && r &&  // (not for a replayable step: its keep vector changes between replays)
        sel->keep_mask_dev && sel->keep_mask_dev >= r->mask_buf && sel->keep_mask_dev < r->mask_buf + 4u * r->mask_stride &&
        (size_t)(sel->keep_mask_dev - r->mask_buf) % r->mask_stride == 0) {
        // a keep vector that came through dmi_set_keep_mask: the host knows what it holds, so
        // admission and accounting work with the record's real size instead of the bound
        const std::vector<uint8_t> &hm = r->mask_host[(size_t)(sel->keep_mask_dev - r->mask_buf) / r->mask_stride];
        if (hm.size() == sel->n_reqs) {
            uint64_t kept = 0;
            for (uint32_t i = 0; i < sel->n_reqs; i++) kept += hm[i] ? sel->reqs[i].tok_count : 0u;
            pl.ub = dmi_record_bytes(sel->n_reqs, kept, geo.row_elems, xf->out_dtype, xf->summary_mask);
            pl.rows_known = kept;
            pl.size_known = true;
        }
    }

    const bool index_mode = sel->row_index_dev != nullptr;
    bool one_row_each = true;
    for (uint32_t i = 0; one_row_each && i < sel->n_reqs; i++) one_row_each = sel->reqs[i].tok_count == 1u;
    const bool simple = one_row_each && sel->keep_mask_dev == nullptr;
    a.rows_known = pl.size_known ? 1u : 0u;
    a.kept_rows = (uint32_t)pl.rows_known;
    a.one_row_each = one_row_each ? 1u : 0u;
    a.listed_rows = (uint32_t)listed;
    const bool tab_lds = !simple && sel->n_reqs <= kLdsTableMax;
    a.n_seg = geo.n_seg;
    a.keep_mask = sel->keep_mask_dev;
    a.row_index = sel->row_index_dev;
    a.n_reqs = sel->n_reqs;
    a.src_dtype = geo.src_dtype;
    a.out_dtype = xf->out_dtype;
    a.summary_mask = xf->summary_mask;
    a.rec_flags = (a.paged ? DMI_REC_PAGED : 0u) | (sel->keep_mask_dev ? DMI_REC_MASKED : 0u) |
                  (index_mode ? DMI_REC_INDEXED : 0u);
    a.row_elems = geo.row_elems;
    a.units_per_row = (uint32_t)upr;
    a.row_lanes = 0;
    if (xf->summary_mask) {                     // as few lanes to a row as four loads each allow
        a.row_lanes = upr > 1024u ? 256u : upr > 256u ? 64u * (uint32_t)((upr + 255u) / 256u) : 4u;
        while (upr <= 256u && 4u * a.row_lanes < upr) a.row_lanes *= 2u;
    }
    a.point_id = point_id;
    a.rank_tag = env.rank_tag;
    a.ring = env.ring;
    a.cap = env.cap;
    a.ctrl = env.ctrl;
    a.simple = simple ? 1u : 0u;
    auto shift_of = [](uint64_t v) { return v && (v & (v - 1u)) == 0 ? (uint32_t)__builtin_ctzll(v) : 32u; };
    a.upr_shift = shift_of(upr);
    a.bs_shift = shift_of(a.block_size);
    a.seg_shift = shift_of(a.seg_units);
    a.table_in_lds = tab_lds ? 1u : 0u;
    a.lds_bytes = capture_lds_bytes(simple ? 0u : sel->n_reqs, index_mode, tab_lds);

    pl.grid = plan_grid(a, 1u);

    // requests listing several rows take the decode-shaped kernel with one workgroup per listed
    // row: a launch whose row count must be able to change later (a replayable step) does not
    pl.decode = decode_kernel_applies(a, geo.vec16) && (one_row_each || fixed_row_count_ok);
    pl.row_map = pl.decode && !one_row_each && !index_mode;
    // (in a replayable step only where dmi_step_update() keeps it so)
    if ((pl.decode || fixed_row_count_ok) && !index_mode && one_row_each && sel->n_reqs) {
        a.rows_consecutive = 1u;
        a.row_first = sel->reqs[0].row_base + sel->reqs[0].tok_start;
        for (uint32_t i = 1; a.rows_consecutive && i < sel->n_reqs; i++)
            a.rows_consecutive = sel->reqs[i].row_base + sel->reqs[i].tok_start == a.row_first + i;
    }
    if (pl.decode) {
        // the host knows this record exactly: geometry and header travel as kernel arguments
        // (the kernel itself puts sequence number and step id into the header)
        const uint64_t table_bytes = pad64((uint64_t)sel->n_reqs * 16u);
        a.payload_bytes = listed * geo.row_elems * dtype_size(xf->out_dtype);
        a.off_payload = DMI_HEADER_BYTES + table_bytes;
        a.off_sum = a.off_payload + pad64(a.payload_bytes);
        a.sum_arr = pad64(listed * 4u);
        a.record_bytes = ub;
        a.hdr[0] = DMI_MAGIC;
        a.hdr[1] = 1u | (DMI_HEADER_BYTES << 16);
        a.hdr[6] = point_id;
        a.hdr[7] = a.src_dtype | (a.out_dtype << 8) | (a.summary_mask << 16) | (a.rec_flags << 24);
        a.hdr[8] = sel->n_reqs;  a.hdr[9] = (uint32_t)listed;  a.hdr[10] = geo.row_elems;  a.hdr[11] = a.rank_tag;
        a.hdr[12] = (uint32_t)ub;               a.hdr[13] = (uint32_t)(ub >> 32);
        a.hdr[14] = (uint32_t)a.payload_bytes;  a.hdr[15] = (uint32_t)(a.payload_bytes >> 32);
    }
    return DMI_OK;
}

// While captures run, a flush by the producer's thread copies no fewer bytes at a time than this, of as many in all.
static uint64_t least_chunk(uint64_t all) { return std::min(std::max(all / 8u, kLeastChunk), 16u * kLeastChunk); }

// Tensors of a batch's first launch where two launches reach the host sooner than one: the flush behind them copies what
// the first has captured (the second's note says so) while the second runs.  A batch of which both the capture and the way over
// the link take long is cut where the first part is across as the second has been captured, at the earliest where a flush takes notice.
// (Only where the ring's last dmi_drain was such a flush, or there has been none: to a drain by another thread, which follows the events, two
// launches are no use, and they cost a launch and the end and the start of a kernel, 10 us of 58 on the producer's stream.)
// That saves capture * link / (capture + link) at best; it costs the launch, and the end and the start of a kernel, and has to be worth 25 us and
// a sixteenth of both together.
// (Saved at best, then one launch / two, delivered, with the tensors in front in brackets, us.  Worth it: 8 caches, 298 MB, norm and largest magnitude
// 33, 155 / 138 (3: 142, 4: 138, 5: 146, 6: 156; in launches of four, three, two, one each 138, 142, 144, 154); 16 such caches 65, 305 / 243; 8 of 514 MB,
// three statistics 65, 339 / 284.  Not worth 25 us: 8 caches, 298 MB, norms alone 23, 112 / 114 (6) to 121 (2); 4 caches, 149 MB 16, 88 / 92 (3) to 94 (2);
// 32 x 256 x 4096 raw 12, 1247 / 1231 (8) to 1240 (24), to fp8 644 / 642 (8) to 649 (24); 80 x 256 x 8192, statistics 9, 79 / 82 (40); 32 x 64 x 4096 raw 3,
// 336 / 334 (24) to 343 (16).  Not a sixteenth: 8 caches raw, 298 MB 53, 5364 / 5302 (2) to 5341 (6), in eight launches 5290: what is
// to be had of a flush that is nearly all link is 1 %.)
static uint32_t first_launch(const CaptureArgs &a, uint64_t ub, uint32_t n)
{
    constexpr uint64_t kReadRate = 5500, kLinkRate = 57;        // bytes per ns
    constexpr uint64_t kWorthNs = 25000;
    const uint64_t rows = a.rows_known ? a.kept_rows : a.listed_rows, all = n * ub;
    const uint64_t capture = n * rows * a.row_elems * dtype_size(a.src_dtype) / kReadRate, link = all / kLinkRate;      // ns
    const uint64_t both = capture + link;
    if (n < 2u || capture * link < std::max(kWorthNs, both / 16u) * both) return n;
    const uint64_t part = all / 1000u * (capture * 1000u / both), least = std::max(least_chunk(all), kWorthNotes);
    if ((n - 1u) * ub < least) return n;
    return (uint32_t)std::min<uint64_t>((std::max(part, least) + ub - 1u) / ub, n - 1u);
}

// Issue the captures of `n` tensors of one shape that share selection and transform (n = 1: an
// ordinary observe): as few launches as the ring and kMaxBatch allow, or one more (first_launch()), each of them producing
// the records, sequence numbers and counters that single launches in the same order would.
// points / srcs list the tensors that passed the gate; *n_launched counts how many of them
// have been issued when the call returns (all of them unless it fails).
dmi_status_t observe_common(dmi_ring *r, uint32_t n, const uint32_t *points, const uint8_t *const *srcs,
                            const dmi_selection_t *sel, const dmi_transform_t *xf, uint64_t step_id,
                            void *hip_stream, const Geometry &geo, CaptureArgs &a, uint32_t *n_launched)
{
    hipStream_t s = (hipStream_t)hip_stream;
    *n_launched = 0;
    if (r->step_open)
        return fail(DMI_ERR_INVALID_ARG, "a replayable step is between dmi_step_begin and dmi_step_end");
    Plan pl;
    dmi_status_t st = plan_capture(plan_env(r), points[0], sel, xf, geo, a, pl, true);
    if (st != DMI_OK) return st;
    const uint64_t ub = pl.ub;
    const uint32_t mode = r->mode.load(std::memory_order_relaxed);
    note_producer(r, hip_stream);
    // a launch of several records lays them down one behind the other from one head: under the
    // completeness policy they must fit the ring together (the kernels rely on it), so a batch
    // that does not is issued in pieces, each waiting for its room as single observes would
    const uint64_t fit = r->dev_cap / ub < kMaxBatch ? r->dev_cap / ub : kMaxBatch;
    // (for a flush that copies by notes, if the ring is flushed like that)
    const bool by_notes = r->notes && r->flushed_by_notes.load(std::memory_order_relaxed);
    const uint32_t n_first = by_notes && mode == DMI_POLICY_BLOCK ? first_launch(a, ub, n) : n;
    uint32_t slot = 0;
    bool staged = false, host_decides = false;
    BatchArgs b;
    memset(&b, 0, sizeof b);

    // one launch: records [first, first + cnt) of the caller's list; force_drop: they are records
    // the host already knows cannot fit, launched with one workgroup each only to be counted; tail:
    // as many records behind the cnt launched ones that the host knows cannot fit either, counted
    // by the same launch without any workgroup of their own
    auto issue = [&](uint32_t first, uint32_t cnt, uint64_t floor, bool force_drop, uint32_t tail) -> dmi_status_t {
        dmi_status_t rc;
        if ((rc = commit_slot_room(r, cnt + tail)) != DMI_OK) return rc;
        if (!staged) {
            if ((rc = stage_selection(r, sel, a.paged != 0, pl.row_map, s, &slot)) != DMI_OK) return rc;
            staged = true;
        }
        const uint64_t seq = r->next_seq.load(std::memory_order_relaxed);
        a.req_table = reinterpret_cast<const uint4 *>(r->slab + (size_t)slot * r->slab_slot_words);
        a.row0 = r->slab + (size_t)slot * r->slab_slot_words + 4u * (size_t)sel->n_reqs;
        a.row_map = pl.row_map ? a.row0 + sel->n_reqs : nullptr;
        a.seq = seq;
        a.n_batch = cnt;
        a.step_id = step_id;
        a.cslot = &r->dctrl->slots[(seq + cnt + tail - 1u) % kCommitSlots];
        a.tail_floor = floor;
        a.drop_newest = mode == DMI_POLICY_DROP_NEWEST ? 1u : 0u;
        a.force_drop = force_drop ? 1u : 0u;
        a.n_tail_drop = tail;
        // best effort: every fourth launch refreshes the drained-up-to mark from the host's word
        // (a read across the host link by one lane); in between, the launch-time floor stands
        a.tail_src = (a.drop_newest && (r->launches.load(std::memory_order_relaxed) & 3u) == 0) ? r->htail_dev : nullptr;
        a.par_in = r->chain_par;
        a.step = nullptr;
        a.node = 0;
        a.note = r->notes && r->unnoted_bytes >= kNoteBytes ? r->hwords_dev + kWordNote : nullptr;
        for (uint32_t i = 0; i < cnt; i++) b.src[i] = srcs[first + i];
        for (uint32_t i = 0; i < cnt + tail; i++) b.point[i] = points[first + i];

        // (only the general kernel counts a tail)
        const bool decode = !force_drop && !tail && pl.decode && batch_takes_decode_kernel(a, cnt);
        const uint32_t grid = force_drop ? 1u : plan_grid(a, cnt, n_first < n ? n : cnt);
        const hipError_t e = decode ? launch_capture_decode(a, b, s) : launch_capture(a, b, grid, geo.vec16, s);
        if (e != hipSuccess) return fail(DMI_ERR_HIP, "capture launch failed: %s", hipGetErrorString(e));
        const uint64_t bytes = force_drop ? 0u : ub * cnt;      // what the launch may add to the ring
        // can the host tell what this launch does?  Under the completeness policy nothing is dropped;
        // under best effort the caller of this function has decided (host_decides) which records fit
        const bool exact = pl.size_known && (mode == DMI_POLICY_BLOCK || host_decides);
        r->chain_par ^= 1u;
        r->last_launch_ns.store(now_ns(), std::memory_order_relaxed);
        {
            std::lock_guard<std::mutex> lk(r->pmu);
            r->launches.fetch_add(1, std::memory_order_relaxed);
            r->next_seq.store(seq + cnt + tail, std::memory_order_release);
            if (exact && !force_drop) {
                r->window.bytes += bytes; r->window.records += cnt; r->window.rows += pl.rows_known * cnt;
                r->window.drop_bytes += ub * tail; r->window.drop_records += tail;
                r->window.drop_rows += pl.rows_known * tail;
            } else if (exact) {
                r->window.drop_bytes += ub * (cnt + tail); r->window.drop_records += cnt + tail;
                r->window.drop_rows += pl.rows_known * (cnt + tail);
            } else {
                r->window_exact = false;
            }
        }
        if (exact && r->head_exact) r->exact_head += bytes;
        else r->head_exact = false;
        r->inflight.emplace_back(seq + cnt + tail - 1u, bytes);    // confirmed launch by launch: the last record stands for all
        r->inflight_sum += bytes;
        r->unprobed_launches += 1;
        r->unprobed_bytes += bytes;
        if (a.note) r->unnoted_bytes = 0;
        r->unnoted_bytes += bytes;
        return DMI_OK;
    };

    for (uint32_t done = 0; done < n;) {
        uint32_t nb = n - done < kMaxBatch ? n - done : kMaxBatch;
        uint32_t n_keep = nb;
        if (mode == DMI_POLICY_BLOCK) {
            if (nb > fit) nb = (uint32_t)fit;
            if (!done && nb > n_first) nb = n_first;
            n_keep = nb;
            if ((st = wait_for_room(r, ub * nb)) != DMI_OK) return st;
        } else {
            head_upper_bound(r);    // keeps the in-flight list short
        }
        const uint64_t floor = r->drain_done.load(std::memory_order_acquire);
        host_decides = false;
        if (mode == DMI_POLICY_DROP_NEWEST && pl.size_known) {
            // Best effort: while the host knows where the head will stand when this launch runs, it
            // knows which records fit, because the kernel decides on this very drained mark or a newer
            // one (a newer one only makes more room).  It then launches the records that fit as
            // usual and the ones that do not apart, with a single workgroup each, only to be counted:
            // under sustained overload those are a third or more of all records, and a full grid of
            // workgroups for each of them, all finding out that they have nothing to do, costs a
            // quarter of what copying the record would.  And since the outcome is known, the host
            // needs no commit slot fetched to follow the head (an event behind the launches will do).
            // Not while the host runs far ahead of the GPU, though: the drained mark it decides on is
            // the one of this moment, the kernel's is at most a launch or so older than its own start.
            if ((st = advance_commits(r, false)) != DMI_OK) return st;
            if (!r->head_exact &&
                r->confirmed.load(std::memory_order_acquire) == r->next_seq.load(std::memory_order_relaxed)) {
                r->head_exact = true;
                r->exact_head = r->committed.load(std::memory_order_acquire);
            }
            constexpr uint64_t kTightLaunches = 4;
            const bool tight = r->launches.load(std::memory_order_relaxed) -
                               r->confirmed_launches.load(std::memory_order_acquire) <= kTightLaunches;
            if (r->head_exact && tight) {
                host_decides = true;
                const uint64_t used = r->exact_head - floor;
                const uint64_t room = used < r->dev_cap ? (r->dev_cap - used) / ub : 0u;
                if (room < nb) n_keep = (uint32_t)room;
            }
        }
        // (a tail is only ever the host's own decision: sizes known, so the launch's outcome is exact)
        // (nothing fits: one workgroup counts them all)
        if (n_keep) st = issue(done, n_keep, floor, false, nb - n_keep);
        else st = issue(done, 1u, floor, true, nb - 1u);
        if (st != DMI_OK) return st;
        done += nb;
        *n_launched = done;
        if (r->unprobed_launches >= 16u || r->unprobed_bytes >= r->probe_bytes) {
            r->unprobed_launches = 0;
            r->unprobed_bytes = 0;
            if ((st = record_probe(r)) != DMI_OK) return st;
        }
    }
    return DMI_OK;
}

// Common front gate: argument checks shared by all observes.
dmi_status_t gate_args(dmi_ring *r, const dmi_selection_t *sel, const dmi_transform_t *xf, uint32_t src_dtype)
{
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    if (!sel || !xf) return fail(DMI_ERR_INVALID_ARG, "selection / transform is NULL");
    if (sel->n_reqs > r->max_reqs)
        return fail(DMI_ERR_INVALID_ARG, "n_reqs %u exceeds max_reqs_per_observe %u", sel->n_reqs, r->max_reqs);
    if (sel->n_reqs && !sel->reqs) return fail(DMI_ERR_INVALID_ARG, "reqs is NULL");
    if (!transform_ok(src_dtype, xf->out_dtype))
        return fail(DMI_ERR_INVALID_ARG, "unsupported dtype pair %u -> %u", src_dtype, xf->out_dtype);
    if (xf->summary_mask & ~7u) return fail(DMI_ERR_INVALID_ARG, "bad summary_mask %u", xf->summary_mask);
    return DMI_OK;
}

// Hook filtering and sampling for one observation (arguments already checked).
// Returns DMI_OK to proceed, a positive code to stop without error.
dmi_status_t gate_point(dmi_ring *r, uint32_t point_id, const dmi_selection_t *sel, uint64_t step_id)
{
    r->observed_calls++;
    if (r->point_off[point_id]) { r->disabled_calls++; return DMI_POINT_DISABLED; }
    const uint32_t k = r->sample_k.load(std::memory_order_relaxed);
    if (step_id % k != r->sample_phase.load(std::memory_order_relaxed)) {
        uint64_t listed = 0;
        for (uint32_t i = 0; i < sel->n_reqs; i++) listed += sel->reqs[i].tok_count;
        r->sampled_out_calls++;
        r->sampled_out_rows += listed;
        return DMI_SAMPLED_OUT;
    }
    return DMI_OK;
}

dmi_status_t gate(dmi_ring *r, uint32_t point_id, const dmi_selection_t *sel, const dmi_transform_t *xf,
                  uint64_t step_id, uint32_t src_dtype)
{
    dmi_status_t st = gate_args(r, sel, xf, src_dtype);
    if (st != DMI_OK) return st;
    if (point_id >= DMI_MAX_POINTS) return fail(DMI_ERR_INVALID_ARG, "point_id %u >= %u", point_id, DMI_MAX_POINTS);
    return gate_point(r, point_id, sel, step_id);
}

// The gate for a batch: every tensor passes it on its own, in order, exactly as if it had been
// observed alone.  live[] receives the positions that go on to be captured.
dmi_status_t gate_batch(dmi_ring *r, uint32_t n, const uint32_t *point_ids, const void *const *data,
                        const dmi_selection_t *sel, const dmi_transform_t *xf, uint64_t step_id, uint32_t src_dtype,
                        std::vector<uint32_t> &live, dmi_status_t *all_stopped)
{
    dmi_status_t st = gate_args(r, sel, xf, src_dtype);
    if (st != DMI_OK) return st;
    if (n && (!point_ids || !data)) return fail(DMI_ERR_INVALID_ARG, "point_ids / data is NULL");
    for (uint32_t i = 0; i < n; i++)
        if (point_ids[i] >= DMI_MAX_POINTS)
            return fail(DMI_ERR_INVALID_ARG, "point_ids[%u] = %u >= %u", i, point_ids[i], DMI_MAX_POINTS);
    live.clear();
    *all_stopped = DMI_POINT_DISABLED;
    for (uint32_t i = 0; i < n; i++) {
        const dmi_status_t g = gate_point(r, point_ids[i], sel, step_id);
        if (g == DMI_OK) live.push_back(i);
        else if (g == DMI_SAMPLED_OUT) *all_stopped = DMI_SAMPLED_OUT;
    }
    return DMI_OK;
}

// The library's drain thread (section 4.3): follows the commits and issues a batch of copies once
// enough has accumulated by any of four measures: committed bytes, committed records, how full the
// device ring is, how long the oldest waiting byte has waited.
void bg_loop(dmi_ring *r)
{
    (void)hipSetDevice(r->dev);
    const uint64_t min_bytes = r->cfg.bg_min_bytes ? r->cfg.bg_min_bytes : (1u << 20);
    const uint64_t min_records = r->cfg.bg_min_records ? r->cfg.bg_min_records : 64u;
    const uint64_t occupancy_pct = r->cfg.bg_occupancy_pct ? r->cfg.bg_occupancy_pct : 50u;
    const uint64_t timeout_ns = (uint64_t)(r->cfg.bg_timeout_us ? r->cfg.bg_timeout_us : 200u) * 1000ull;
    // how long the producer must have paused before this thread puts a probe of its own behind
    // its launches (while it keeps launching it probes by itself)
    const uint64_t quiet_ns = timeout_ns < 200000ull ? timeout_ns : 200000ull;
    uint64_t waiting_since = 0, last_probe = 0;
    while (!r->stop.load(std::memory_order_acquire)) {
        if (r->quiet.load(std::memory_order_acquire)) {
            // a stream capture is open on the producer's side: stay away from the HIP API
            r->bg_parked.store(true, std::memory_order_release);
            std::this_thread::sleep_for(std::chrono::microseconds(50));
            continue;
        }
        r->bg_parked.store(false, std::memory_order_release);
        bool idle_probes;
        {
            std::lock_guard<std::mutex> lk(r->pmu);
            idle_probes = r->probes.empty();
        }
        // every probe is a barrier, or a small launch, in the inference queue
        if (idle_probes && now_ns() - last_probe >= quiet_ns &&
            now_ns() - r->last_launch_ns.load(std::memory_order_relaxed) >= quiet_ns) {
            (void)record_probe(r);
            last_probe = now_ns();
        }
        (void)advance_commits(r, false);
        uint64_t pending_bytes, pending_records, undrained;
        {
            std::lock_guard<std::mutex> lk(r->mu);
            // copies issued by somebody's non-blocking dmi_drain are noted here as they finish: with
            // this thread running, nobody else looks at the drain stream
            (void)reap(r);
            uint64_t committed, committed_records;
            {
                std::lock_guard<std::mutex> pk(r->pmu);
                committed = read_committed(r);
                committed_records = r->snap[0];
            }
            pending_bytes = committed - r->drain_issued;
            pending_records = pending_bytes ? committed_records - r->drain_issued_records : 0u;
            undrained = committed - r->drain_done.load(std::memory_order_relaxed);
        }
        const uint64_t t = now_ns();
        if (pending_bytes == 0) waiting_since = 0;
        else if (!waiting_since) waiting_since = t;
        const bool by_bytes = pending_bytes >= min_bytes;
        const bool by_records = pending_records >= min_records;
        const bool by_occupancy = pending_bytes && undrained * 100u >= occupancy_pct * r->dev_cap;
        const bool by_timeout = pending_bytes && t - waiting_since >= timeout_ns;
        if (by_bytes || by_records || by_occupancy || by_timeout) {
            uint64_t moved = 0;
            (void)drain(r, true, &moved);
            waiting_since = 0;
            if (moved) continue;
        }
        std::this_thread::sleep_for(std::chrono::microseconds(20));
    }
}

void free_ring(dmi_ring *r)
{
    if (!r) return;
    if (r->drain_stream) { (void)hipStreamSynchronize(r->drain_stream); (void)hipStreamDestroy(r->drain_stream); }
    if (r->ctl_stream) { (void)hipStreamSynchronize(r->ctl_stream); (void)hipStreamDestroy(r->ctl_stream); }
    if (r->hwords) (void)hipHostFree(r->hwords);
    for (auto &p : r->probes) if (p.ev) (void)hipEventDestroy(p.ev);
    for (auto ev : r->probe_pool) (void)hipEventDestroy(ev);
    if (r->dev_ring) (void)hipFree(r->dev_ring);
    if (r->dctrl) (void)hipFree(r->dctrl);
    if (r->slab) (void)hipFree(r->slab);
    if (r->mask_buf) (void)hipFree(r->mask_buf);
    if (r->host_ring) (void)hipHostFree(r->host_ring);
    if (r->hslots) (void)hipHostFree((void *)r->hslots);
    delete r;
}


}  // namespace host
}  // namespace dmi

// =========================================================================== C ABI
extern "C" {

const char *dmi_last_error(void) { return last_error_cstr(); }
const char *dmi_version(void) { return "dmi-ring 0.1 (gfx950)"; }

#ifndef DMI_HEADER_DIGEST
#define DMI_HEADER_DIGEST 0
#endif
uint64_t dmi_debug_header_digest(void) { return DMI_HEADER_DIGEST; }

uint64_t dmi_record_bytes(uint32_t n_reqs, uint64_t n_rows, uint32_t row_elems, uint32_t out_dtype,
                          uint32_t summary_mask)
{
    uint64_t b = DMI_HEADER_BYTES;
    b += pad64((uint64_t)n_reqs * 16u);
    b += pad64(n_rows * row_elems * dtype_size(out_dtype));
    b += (uint64_t)__builtin_popcount(summary_mask & 7u) * pad64(n_rows * 4u);
    return b;
}

dmi_status_t dmi_ring_create(const dmi_ring_config_t *cfg, dmi_ring_t **out)
{
    if (!cfg || !out) return fail(DMI_ERR_INVALID_ARG, "cfg / out is NULL");
    if (cfg->device_ring_bytes < 4096 || cfg->host_ring_bytes < 4096 || cfg->device_ring_bytes % 64 ||
        cfg->host_ring_bytes % 64)
        return fail(DMI_ERR_INVALID_ARG, "ring sizes must be multiples of 64 and at least 4096");
    if ((cfg->flags & DMI_DRAIN_COPY_ENGINE) && (cfg->flags & DMI_DRAIN_KERNEL))
        return fail(DMI_ERR_INVALID_ARG, "choose one drain mode");
    // DMI_DRAIN_MODE=kernel|copy in the environment overrides the drain engine (for comparisons
    // without touching the caller's code)
    uint32_t flags = cfg->flags;
    if (const char *m = getenv("DMI_DRAIN_MODE")) {
        if (!strcmp(m, "kernel")) flags = (flags & ~(uint32_t)DMI_DRAIN_COPY_ENGINE) | DMI_DRAIN_KERNEL;
        else if (!strcmp(m, "copy")) flags = (flags & ~(uint32_t)DMI_DRAIN_KERNEL) | DMI_DRAIN_COPY_ENGINE;
        else return fail(DMI_ERR_INVALID_ARG, "DMI_DRAIN_MODE must be 'kernel' or 'copy'");
    }
    const uint32_t max_reqs = cfg->max_reqs_per_observe ? cfg->max_reqs_per_observe : 1024u;
    if (max_reqs > 4096u) return fail(DMI_ERR_INVALID_ARG, "max_reqs_per_observe > 4096");
    int n_dev = 0;
    hipError_t e = hipGetDeviceCount(&n_dev);
    if (e != hipSuccess || n_dev <= 0)
        return fail(DMI_ERR_HIP, "no HIP device available (%s)", hipGetErrorString(e));
    if (cfg->device_id < 0 || cfg->device_id >= n_dev) return fail(DMI_ERR_INVALID_ARG, "bad device_id");
    HIP_TRY(hipSetDevice(cfg->device_id));

    dmi_ring *r = new (std::nothrow) dmi_ring;
    if (!r) return fail(DMI_ERR_NOMEM, "out of host memory");
    r->cfg = *cfg;
    r->cfg.flags = flags;
    r->dev = cfg->device_id;
    r->dev_cap = cfg->device_ring_bytes;
    r->host_cap = cfg->host_ring_bytes;
    r->max_reqs = max_reqs;
    r->block_timeout_ms = cfg->block_timeout_ms ? cfg->block_timeout_ms : 2000u;
    r->point_off.assign(DMI_MAX_POINTS, 0);
    r->slab_slot_words = (max_reqs * 5u + kDecodeMaxListed + 63u) & ~63u;
    // a probe at least every 16 launches, or every 1/32 of the ring (not under 8 MiB): often enough
    // for the drain to follow closely, rare enough that its cost in the producer's stream stays small
    r->probe_bytes = r->dev_cap / 32u > (8u << 20) ? r->dev_cap / 32u : (8u << 20);

    auto bail = [&](hipError_t err, const char *what) {
        fail(DMI_ERR_HIP, "%s failed: %s", what, hipGetErrorString(err));
        free_ring(r);
        return DMI_ERR_HIP;
    };
    if ((e = hipMalloc((void **)&r->dev_ring, r->dev_cap)) != hipSuccess) return bail(e, "hipMalloc(device ring)");
    if ((e = hipMalloc((void **)&r->dctrl, sizeof(DevCtrl))) != hipSuccess) return bail(e, "hipMalloc(ctrl)");
    if ((e = hipMalloc((void **)&r->slab, (size_t)kSlabSlots * r->slab_slot_words * 4u)) != hipSuccess)
        return bail(e, "hipMalloc(selection slab)");
    r->mask_stride = (max_reqs + 255u) & ~255u;
    if ((e = hipMalloc((void **)&r->mask_buf, (size_t)4u * r->mask_stride)) != hipSuccess)
        return bail(e, "hipMalloc(keep vectors)");
    if ((e = hipHostMalloc((void **)&r->host_ring, r->host_cap, hipHostMallocMapped)) != hipSuccess)
        return bail(e, "hipHostMalloc(host ring)");
    if ((e = hipHostGetDevicePointer((void **)&r->host_ring_dev, r->host_ring, 0)) != hipSuccess)
        return bail(e, "hipHostGetDevicePointer(host ring)");
    // touch every page now: the consumer's first read of a page should not pay for a fault
    memset(r->host_ring, 0, r->host_cap);
    if ((e = hipHostMalloc((void **)&r->hslots, sizeof(CommitSlot) * kCommitSlots,
                           hipHostMallocMapped | hipHostMallocCoherent)) != hipSuccess)
        return bail(e, "hipHostMalloc(commit slots)");
    if ((e = hipHostGetDevicePointer((void **)&r->hslots_dev, (void *)r->hslots, 0)) != hipSuccess)
        return bail(e, "hipHostGetDevicePointer(commit slots)");
    memset((void *)r->hslots, 0, sizeof(CommitSlot) * kCommitSlots);
    {
        DevCtrl *init = new (std::nothrow) DevCtrl;
        if (!init) { free_ring(r); return fail(DMI_ERR_NOMEM, "out of host memory"); }
        memset(init, 0, sizeof *init);
        e = hipMemcpy(r->dctrl, init, sizeof *init, hipMemcpyHostToDevice);
        delete init;
        if (e != hipSuccess) return bail(e, "hipMemcpy(ctrl)");
    }
    if ((e = hipHostMalloc((void **)&r->hwords, kWords * 8u, hipHostMallocMapped | hipHostMallocCoherent)) != hipSuccess)
        return bail(e, "hipHostMalloc(words)");
    if ((e = hipHostGetDevicePointer((void **)&r->hwords_dev, r->hwords, 0)) != hipSuccess)
        return bail(e, "hipHostGetDevicePointer(words)");
    memset(r->hwords, 0, kWords * 8u);
    r->htail = r->hwords + kWordTail;
    r->htail_dev = r->hwords_dev + kWordTail;
    // Notes, which say that what earlier launches have written can be copied while a later one runs: the release at a launch's end
    // reaches memory, not only L2, where the compute units that the next launch may run on do not share one L2 (32 of them do).
    int units = 0;
    if ((e = hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, r->dev)) != hipSuccess)
        return bail(e, "hipDeviceGetAttribute");
    // And they are for rings that choose their engine, and whose copies nobody but a flush starts.
    r->notes = units > 32 && !(flags & (DMI_BG_THREAD | DMI_DRAIN_COPY_ENGINE | DMI_DRAIN_KERNEL));
    if ((e = hipStreamCreateWithFlags(&r->drain_stream, hipStreamNonBlocking)) != hipSuccess)
        return bail(e, "hipStreamCreate");
    if ((e = hipStreamCreateWithFlags(&r->ctl_stream, hipStreamNonBlocking)) != hipSuccess)
        return bail(e, "hipStreamCreate");
    if ((e = hipDeviceSynchronize()) != hipSuccess) return bail(e, "hipDeviceSynchronize");
    if (flags & DMI_BG_THREAD) r->bg = std::thread(bg_loop, r);
    *out = r;
    return DMI_OK;
}

dmi_status_t dmi_ring_destroy(dmi_ring_t *r)
{
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    (void)hipSetDevice(r->dev);
    (void)dmi_exporter_stop(r);
    r->stop.store(true, std::memory_order_release);
    if (r->bg.joinable()) r->bg.join();
    free_ring(r);
    return DMI_OK;
}

}  // extern "C"

namespace dmi {
namespace host {

// Checks of a selection against a dense source of T rows (not in index mode, where the
// kernel checks every index itself).
dmi_status_t check_dense_rows(const dmi_req_sel_t *reqs, uint32_t n, int64_t T)
{
    for (uint32_t i = 0; i < n; i++) {
        const dmi_req_sel_t &q = reqs[i];
        if (!q.tok_count) continue;
        const uint64_t last = (uint64_t)q.row_base + q.tok_start + (uint64_t)(q.tok_count - 1u) * q.tok_step;
        if (last >= (uint64_t)T)
            return fail(DMI_ERR_INVALID_ARG, "request %u selects row %llu of a %lld-row tensor", i,
                        (unsigned long long)last, (long long)T);
    }
    return DMI_OK;
}

// Same for a paged source: block-table row and token positions.
dmi_status_t check_paged_rows(const dmi_req_sel_t *reqs, uint32_t n, uint32_t n_seqs, uint32_t block_size,
                              int64_t bt_stride)
{
    for (uint32_t i = 0; i < n; i++) {
        const dmi_req_sel_t &q = reqs[i];
        if (q.row_base >= n_seqs) return fail(DMI_ERR_INVALID_ARG, "request %u: block-table row out of range", i);
        if (!q.tok_count) continue;
        const uint64_t last = (uint64_t)q.tok_start + (uint64_t)(q.tok_count - 1u) * q.tok_step;
        if (last > 0x7FFFFFFFull || last / block_size >= (uint64_t)bt_stride)
            return fail(DMI_ERR_INVALID_ARG, "request %u: token %llu is beyond the block table", i,
                        (unsigned long long)last);
    }
    return DMI_OK;
}

// Validate a dense tensor + selection and fill the source part of the kernel arguments.
dmi_status_t prep_dense(const dmi_tensor_t *t, const dmi_selection_t *sel, Geometry &geo, CaptureArgs &a)
{
    const uint32_t es = dtype_size(t->dtype);
    const int64_t T = t->shape[0], E = t->shape[1];
    if (T < 0 || T > 0xFFFFFFFFll || E < 1 || E > 0x7FFFFFFF) return fail(DMI_ERR_INVALID_ARG, "bad tensor shape");
    if ((E > 1 && t->stride[1] != 1) || t->stride[0] < 0) return fail(DMI_ERR_INVALID_ARG, "bad tensor stride");
    if (!t->data && T > 0) return fail(DMI_ERR_INVALID_ARG, "tensor data is NULL");
    if ((uintptr_t)t->data % es) return fail(DMI_ERR_INVALID_ARG, "tensor data is not element aligned");
    if (!sel->row_index_dev) {
        dmi_status_t st = check_dense_rows(sel->reqs, sel->n_reqs, T);
        if (st != DMI_OK) return st;
    }
    geo.src_dtype = t->dtype;
    geo.row_elems = (uint32_t)E;
    geo.n_seg = 1;
    geo.seg_elems = (uint32_t)E;
    geo.vec16 = (uintptr_t)t->data % 16 == 0 && ((uint64_t)t->stride[0] * es) % 16 == 0 && ((uint64_t)E * es) % 16 == 0;
    memset(&a, 0, sizeof a);
    a.src = (const uint8_t *)t->data;
    a.row_stride_b = t->stride[0] * (int64_t)es;
    a.n_src_rows = T;
    a.paged = 0;
    a.block_size = 1;
    return DMI_OK;
}

// Validate a paged KV description + selection and fill the source part of the kernel arguments.
dmi_status_t prep_paged(const dmi_paged_kv_t *kv, const dmi_selection_t *sel, Geometry &geo, CaptureArgs &a)
{
    const uint32_t es = dtype_size(kv->dtype);
    if (sel->row_index_dev) return fail(DMI_ERR_INVALID_ARG, "row_index_dev is not valid for paged captures");
    if (!kv->base || !kv->block_table_dev) return fail(DMI_ERR_INVALID_ARG, "kv base / block table is NULL");
    if (!kv->block_size || !kv->head_dim || !kv->n_heads || !kv->n_blocks || !kv->n_seqs)
        return fail(DMI_ERR_INVALID_ARG, "kv geometry has a zero field");
    if (kv->n_heads_sel < 1 || kv->n_heads_sel > DMI_MAX_HEADS_SEL)
        return fail(DMI_ERR_INVALID_ARG, "n_heads_sel must be 1..%u", DMI_MAX_HEADS_SEL);
    for (uint32_t i = 0; i < kv->n_heads_sel; i++)
        if (kv->heads_sel[i] >= kv->n_heads) return fail(DMI_ERR_INVALID_ARG, "selected head out of range");
    if (kv->block_stride < 0 || kv->slot_stride < 0 || kv->head_stride < 0 || kv->block_table_stride < 1)
        return fail(DMI_ERR_INVALID_ARG, "negative kv stride");
    if ((uintptr_t)kv->base % es) return fail(DMI_ERR_INVALID_ARG, "kv base is not element aligned");
    if ((uint64_t)kv->n_heads_sel * kv->head_dim > 0x7FFFFFFFull) return fail(DMI_ERR_INVALID_ARG, "row too long");
    {
        dmi_status_t st = check_paged_rows(sel->reqs, sel->n_reqs, kv->n_seqs, kv->block_size, kv->block_table_stride);
        if (st != DMI_OK) return st;
    }
    geo.src_dtype = kv->dtype;
    geo.n_seg = kv->n_heads_sel;
    geo.seg_elems = kv->head_dim;
    geo.row_elems = kv->n_heads_sel * kv->head_dim;
    geo.vec16 = (uintptr_t)kv->base % 16 == 0 && ((uint64_t)kv->block_stride * es) % 16 == 0 &&
                ((uint64_t)kv->slot_stride * es) % 16 == 0 && ((uint64_t)kv->head_stride * es) % 16 == 0 &&
                ((uint64_t)kv->head_dim * es) % 16 == 0;
    memset(&a, 0, sizeof a);
    a.src = (const uint8_t *)kv->base;
    a.n_src_rows = kv->n_blocks;
    a.block_stride_b = kv->block_stride * (int64_t)es;
    a.slot_stride_b = kv->slot_stride * (int64_t)es;
    a.head_stride_b = kv->head_stride * (int64_t)es;
    a.block_table = kv->block_table_dev;
    a.bt_stride = kv->block_table_stride;
    a.block_size = kv->block_size;
    for (uint32_t i = 0; i < kv->n_heads_sel; i++) a.heads_sel[i] = kv->heads_sel[i];
    a.paged = 1;
    return DMI_OK;
}

}  // namespace host
}  // namespace dmi

extern "C" {

dmi_status_t dmi_observe(dmi_ring_t *r, uint32_t point_id, const dmi_tensor_t *t, const dmi_selection_t *sel,
                         const dmi_transform_t *xf, uint64_t step_id, void *hip_stream)
{
    if (!t) return fail(DMI_ERR_INVALID_ARG, "tensor is NULL");
    dmi_status_t g = gate(r, point_id, sel, xf, step_id, t->dtype);
    if (g != DMI_OK) return g;
    Geometry geo;
    CaptureArgs a;
    if ((g = prep_dense(t, sel, geo, a)) != DMI_OK) return g;
    (void)hipSetDevice(r->dev);
    uint32_t launched = 0;
    return observe_common(r, 1u, &point_id, &a.src, sel, xf, step_id, hip_stream, geo, a, &launched);
}

dmi_status_t dmi_observe_paged(dmi_ring_t *r, uint32_t point_id, const dmi_paged_kv_t *kv,
                               const dmi_selection_t *sel, const dmi_transform_t *xf, uint64_t step_id,
                               void *hip_stream)
{
    if (!kv) return fail(DMI_ERR_INVALID_ARG, "kv is NULL");
    dmi_status_t g = gate(r, point_id, sel, xf, step_id, kv->dtype);
    if (g != DMI_OK) return g;
    Geometry geo;
    CaptureArgs a;
    if ((g = prep_paged(kv, sel, geo, a)) != DMI_OK) return g;
    (void)hipSetDevice(r->dev);
    uint32_t launched = 0;
    return observe_common(r, 1u, &point_id, &a.src, sel, xf, step_id, hip_stream, geo, a, &launched);
}

}  // extern "C"

namespace {

// The batch entry points behind their argument checks: gate every tensor, capture the ones
// that pass.  `first` is the source the geometry was prepared from (its alignment is checked
// with the others here).
dmi_status_t observe_batch(dmi_ring *r, uint32_t n, const uint32_t *point_ids, const void *const *data,
                           const dmi_selection_t *sel, const dmi_transform_t *xf, uint64_t step_id, void *hip_stream,
                           Geometry &geo, CaptureArgs &a, uint32_t *n_done)
{
    std::vector<uint32_t> live;
    dmi_status_t stopped = DMI_OK;
    dmi_status_t g = gate_batch(r, n, point_ids, data, sel, xf, step_id, geo.src_dtype, live, &stopped);
    if (g != DMI_OK) return g;
    if (live.empty()) {
        if (n_done) *n_done = n;
        return n ? stopped : DMI_OK;
    }
    std::vector<uint32_t> pts(live.size());
    std::vector<const uint8_t *> srcs(live.size());
    for (size_t k = 0; k < live.size(); k++) {
        pts[k] = point_ids[live[k]];
        srcs[k] = static_cast<const uint8_t *>(data[live[k]]);
    }
    (void)hipSetDevice(r->dev);
    uint32_t launched = 0;
    g = observe_common(r, (uint32_t)live.size(), pts.data(), srcs.data(), sel, xf, step_id, hip_stream, geo, a,
                       &launched);
    // positions of the caller's arrays dealt with: everything in front of the first tensor not yet issued
    if (n_done) *n_done = launched == live.size() ? n : live[launched];
    return g;
}

}  // namespace

extern "C" {

dmi_status_t dmi_observe_batch(dmi_ring_t *r, uint32_t n, const uint32_t *point_ids, const void *const *data,
                               const dmi_tensor_t *like, const dmi_selection_t *sel, const dmi_transform_t *xf,
                               uint64_t step_id, void *hip_stream, uint32_t *n_done)
{
    if (n_done) *n_done = 0;
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    if (!like) return fail(DMI_ERR_INVALID_ARG, "tensor description is NULL");
    if (!sel || !xf) return fail(DMI_ERR_INVALID_ARG, "selection / transform is NULL");
    if (n && (!point_ids || !data)) return fail(DMI_ERR_INVALID_ARG, "point_ids / data is NULL");
    if (!n) return DMI_OK;
    dmi_tensor_t t = *like;
    t.data = data[0];
    Geometry geo;
    CaptureArgs a;
    dmi_status_t g = prep_dense(&t, sel, geo, a);
    if (g != DMI_OK) return g;
    bool all16 = true;
    if ((g = check_batch_sources(n, data, dtype_size(t.dtype), &all16)) != DMI_OK) return g;
    geo.vec16 = geo.vec16 && all16;
    return observe_batch(r, n, point_ids, data, sel, xf, step_id, hip_stream, geo, a, n_done);
}

dmi_status_t dmi_observe_paged_batch(dmi_ring_t *r, uint32_t n, const uint32_t *point_ids, const void *const *bases,
                                     const dmi_paged_kv_t *like, const dmi_selection_t *sel,
                                     const dmi_transform_t *xf, uint64_t step_id, void *hip_stream, uint32_t *n_done)
{
    if (n_done) *n_done = 0;
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    if (!like) return fail(DMI_ERR_INVALID_ARG, "kv description is NULL");
    if (!sel || !xf) return fail(DMI_ERR_INVALID_ARG, "selection / transform is NULL");
    if (n && (!point_ids || !bases)) return fail(DMI_ERR_INVALID_ARG, "point_ids / bases is NULL");
    if (!n) return DMI_OK;
    dmi_paged_kv_t kv = *like;
    kv.base = bases[0];
    Geometry geo;
    CaptureArgs a;
    dmi_status_t g = prep_paged(&kv, sel, geo, a);
    if (g != DMI_OK) return g;
    bool all16 = true;
    if ((g = check_batch_sources(n, bases, dtype_size(kv.dtype), &all16)) != DMI_OK) return g;
    geo.vec16 = geo.vec16 && all16;
    return observe_batch(r, n, point_ids, bases, sel, xf, step_id, hip_stream, geo, a, n_done);
}

dmi_status_t dmi_drain(dmi_ring_t *r, uint32_t flags, uint64_t *bytes_moved)
{
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    (void)hipSetDevice(r->dev);
    if (bytes_moved) *bytes_moved = 0;
    const bool wait = !(flags & DMI_DRAIN_NONBLOCK);
    const bool by_chunks = (flags & DMI_DRAIN_FLUSH) && r->notes &&
                           r->producer.load(std::memory_order_relaxed) == this_thread();
    r->flushed_by_notes.store(by_chunks, std::memory_order_relaxed);
    dmi_status_t st;
    if (!(flags & DMI_DRAIN_FLUSH)) {
        bool idle_probes;
        {
            std::lock_guard<std::mutex> lk(r->pmu);
            idle_probes = r->probes.empty();
        }
        if (idle_probes && (st = record_probe(r)) != DMI_OK) return st;
        if ((st = advance_commits(r, false)) != DMI_OK) return st;
        if (wait && (st = wait_for_direct(r)) != DMI_OK) return st;
        return drain(r, wait, bytes_moved);
    }
    // flush: everything issued so far must finish, then all of it is moved
    const uint64_t want_seq = r->next_seq.load(std::memory_order_acquire);
    const uint64_t t0 = now_ns();
    uint64_t total = 0, target = UINT64_MAX;
    uint64_t direct = 0;
    if ((st = advance_commits(r, false)) != DMI_OK) return st;
    if ((st = flush_behind_captures(r, &total, &direct)) != DMI_OK) return st;
    if (bytes_moved) *bytes_moved = total;
    if (!direct && (st = record_probe(r)) != DMI_OK) return st;
    // The producer's own thread does not wait for all captures before it copies the first: it polls the notes that they leave, and starts
    // a copy of what is complete as soon as that is worth one (an eighth of it all; every copy costs the link some 8 us).
    ChunkRule rule = {0, true, true, false};
    uint64_t least = 0, last_move = t0;
    if (by_chunks) {
        const uint64_t all = head_upper_bound(r) - r->drain_done.load(std::memory_order_acquire);
        least = least_chunk(all);
    }
    for (;;) {
        if ((st = advance_commits(r, false)) != DMI_OK) return st;
        // once the launches issued before the call are known to have finished, their records lie
        // below the head committed at that moment: the call is done when the drain has passed it,
        // whatever a producer thread commits behind it in the meantime
        if (target == UINT64_MAX && r->confirmed.load(std::memory_order_acquire) >= want_seq)
            target = read_committed(r);
        // (what is complete waits for more of it while there may soon be more)
        rule.more = target == UINT64_MAX;
        const uint64_t idle = now_ns() - last_move;
        rule.least = idle < kChunkPatienceNs ? least : 1u;
        // (what the last copy that the call has started still waits for is the link: no limit applies to it)
        rule.poll = by_chunks && idle < kPollNs;
        uint64_t moved = 0;
        bool host_full = false;
        if ((st = drain(r, true, &moved, &host_full, by_chunks ? &rule : nullptr)) != DMI_OK) return st;
        total += moved;
        if (bytes_moved) *bytes_moved = total;
        if (target != UINT64_MAX && r->drain_done.load(std::memory_order_acquire) >= target) return DMI_OK;
        if (moved) { rule.engine = !rule.more; last_move = now_ns(); continue; }
        if (target != UINT64_MAX && host_full)
            return fail(DMI_ERR_AGAIN, "host ring is full: release records and drain again");
        const uint64_t waited = now_ns() - t0;
        if (direct && waited > kPollNs) {
            if ((st = event_behind(r, direct)) != DMI_OK) return st;
            direct = 0;
        }
        if (waited > (uint64_t)r->block_timeout_ms * 1000000ull && (target == UINT64_MAX || !rule.poll))
            return fail(DMI_ERR_AGAIN, target == UINT64_MAX ? "observes did not finish within %u ms"
                                                            : "the drain did not finish within %u ms",
                        r->block_timeout_ms);
        pause_since(r, last_move);
    }
}

dmi_status_t dmi_poll_host(dmi_ring_t *r, dmi_record_view_t *out, uint32_t max, uint32_t *n)
{
    if (!r || !n || (max && !out)) return fail(DMI_ERR_INVALID_ARG, "NULL argument");
    if (r->exp_running.load()) return fail(DMI_ERR_INVALID_ARG, "the exporter is this ring's consumer");
    return poll_host_impl(r, out, max, n);
}

}  // extern "C"

namespace dmi {
namespace host {
dmi_status_t poll_host_impl(dmi_ring *r, dmi_record_view_t *out, uint32_t max, uint32_t *n)
{
    *n = 0;
    std::lock_guard<std::mutex> lk(r->mu);
    // with the library's drain thread running, arrivals are noted by that thread; a HIP call
    // on the drain stream's events from here would queue up behind its blocking wait
    if (!(r->cfg.flags & DMI_BG_THREAD) && !r->quiet.load(std::memory_order_acquire)) {
        // (the end of a span on the producer's stream is seen by its probe, and only there; a consumer may do nothing but poll)
        dmi_status_t st = r->direct_probe ? advance_commits(r, false) : DMI_OK;
        if (st == DMI_OK) st = reap(r);
        if (st != DMI_OK) return st;
    }
    const uint64_t done = r->drain_done.load(std::memory_order_acquire);
    while (*n < max && r->poll_cursor + DMI_HEADER_BYTES <= done) {
        const uint64_t off = r->poll_cursor % r->host_cap;
        const uint8_t *h = r->host_ring + off;      // capacities and records are multiples of 64
        uint32_t magic;
        uint64_t seq, rb;
        memcpy(&magic, h, 4);
        memcpy(&seq, h + 8, 8);
        memcpy(&rb, h + 48, 8);
        if (magic != DMI_MAGIC || rb < DMI_HEADER_BYTES || rb % 64 || rb > r->dev_cap)
            return fail(DMI_ERR_CLOSED, "corrupt record header at stream offset %llu",
                        (unsigned long long)r->poll_cursor);
        if (r->poll_cursor + rb > done) break;
        dmi_record_view_t &v = out[*n];
        v.p0 = h;
        v.n0 = rb < r->host_cap - off ? rb : r->host_cap - off;
        v.n1 = rb - v.n0;
        v.p1 = v.n1 ? r->host_ring : nullptr;
        v.seq = seq;
        r->polled.emplace_back(seq, r->poll_cursor + rb);
        r->poll_cursor += rb;
        ++*n;
    }
    return DMI_OK;
}

dmi_status_t release_host_impl(dmi_ring *r, uint64_t upto)
{
    std::lock_guard<std::mutex> lk(r->mu);
    while (!r->polled.empty() && r->polled.front().first <= upto) {
        r->released_bytes += r->polled.front().second - r->released;
        r->released = r->polled.front().second;
        r->polled.pop_front();
    }
    return DMI_OK;
}
}  // namespace host
}  // namespace dmi

extern "C" {

dmi_status_t dmi_release_host(dmi_ring_t *r, uint64_t upto)
{
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    if (r->exp_running.load()) return fail(DMI_ERR_INVALID_ARG, "the exporter is this ring's consumer");
    return release_host_impl(r, upto);
}

dmi_status_t dmi_set_policy(dmi_ring_t *r, const dmi_policy_t *p)
{
    if (!r || !p) return fail(DMI_ERR_INVALID_ARG, "NULL argument");
    if (p->mode > DMI_POLICY_DROP_NEWEST || p->sample_k < 1 || p->sample_phase >= p->sample_k)
        return fail(DMI_ERR_INVALID_ARG, "bad policy");
    r->mode.store(p->mode);
    r->sample_k.store(p->sample_k);
    r->sample_phase.store(p->sample_phase);
    return DMI_OK;
}

dmi_status_t dmi_policy_select(uint32_t strategy, const dmi_req_info_t *reqs, uint32_t n, uint64_t bytes_per_row,
                               uint64_t budget, uint8_t *keep, uint32_t *n_kept)
{
    if (strategy > DMI_SELECT_KEEP_BY_PATTERN) return fail(DMI_ERR_INVALID_ARG, "unknown selection strategy");
    if (n && (!reqs || !keep)) return fail(DMI_ERR_INVALID_ARG, "NULL argument");
    std::vector<uint32_t> order(n);
    for (uint32_t i = 0; i < n; i++) order[i] = i;
    const bool by_pattern = strategy == DMI_SELECT_KEEP_BY_PATTERN;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        if (by_pattern) {
            const bool mx = reqs[x].matches != 0, my = reqs[y].matches != 0;
            if (mx != my) return mx;
        }
        return reqs[x].admit_order < reqs[y].admit_order;
    });
    uint64_t used = 0;
    uint32_t kept = 0;
    bool open = true;       // a prefix: once a request does not fit, nothing after it is kept
    for (uint32_t k = 0; k < n; k++) {
        const uint32_t i = order[k];
        const unsigned __int128 cost = (unsigned __int128)reqs[i].rows * bytes_per_row;
        if (open && cost <= (unsigned __int128)(budget - used)) {
            used += (uint64_t)cost;
            keep[i] = 1;
            kept++;
        } else {
            open = false;
            keep[i] = 0;
        }
    }
    if (n_kept) *n_kept = kept;
    return DMI_OK;
}

dmi_status_t dmi_ring_free_bytes(dmi_ring_t *r, uint64_t *free_bytes)
{
    if (!r || !free_bytes) return fail(DMI_ERR_INVALID_ARG, "NULL argument");
    (void)hipSetDevice(r->dev);
    dmi_status_t st = advance_commits(r, false);
    if (st != DMI_OK) return st;
    const uint64_t used = head_upper_bound(r) - r->drain_done.load(std::memory_order_acquire);
    *free_bytes = used < r->dev_cap ? r->dev_cap - used : 0;
    return DMI_OK;
}

dmi_status_t dmi_set_keep_mask(dmi_ring_t *r, const uint8_t *keep, uint32_t n, void *hip_stream,
                               const uint8_t **keep_mask_dev)
{
    if (!r || !keep_mask_dev || (n && !keep)) return fail(DMI_ERR_INVALID_ARG, "NULL argument");
    if (n > r->max_reqs) return fail(DMI_ERR_INVALID_ARG, "n_reqs %u exceeds max_reqs_per_observe %u", n, r->max_reqs);
    (void)hipSetDevice(r->dev);
    const uint32_t which = r->mask_rr++ % 4u;
    uint8_t *dst = r->mask_buf + (size_t)which * r->mask_stride;
    r->mask_host[which].assign(keep, keep + n);
    std::vector<uint32_t> words((n + 3u) / 4u, 0u);
    if (n) memcpy(words.data(), keep, n);
    if (n) HIP_TRY(launch_upload(reinterpret_cast<uint32_t *>(dst), words.data(), (uint32_t)words.size(),
                                 (hipStream_t)hip_stream));
    *keep_mask_dev = dst;
    return DMI_OK;
}

dmi_status_t dmi_point_enable(dmi_ring_t *r, uint32_t point_id, int enabled)
{
    if (!r || point_id >= DMI_MAX_POINTS) return fail(DMI_ERR_INVALID_ARG, "bad ring / point_id");
    r->point_off[point_id] = enabled ? 0 : 1;
    return DMI_OK;
}

dmi_status_t dmi_get_stats(dmi_ring_t *r, dmi_stats_t *o)
{
    if (!r || !o) return fail(DMI_ERR_INVALID_ARG, "NULL argument");
    memset(o, 0, sizeof *o);
    o->observed_calls = r->observed_calls;
    (void)hipSetDevice(r->dev);
    (void)advance_commits(r, false);
    {
        std::lock_guard<std::mutex> lk(r->pmu);
        o->launched_records = r->next_seq.load();       // (with the counters: what has been captured has been launched)
        o->captured_records = r->snap[0];
        o->captured_rows = r->snap[1];
        o->captured_bytes = r->snap[2];
        o->dropped_records = r->snap[3];
        o->dropped_rows = r->snap[4];
        o->dropped_bytes = r->snap[5];
    }
    o->sampled_out_calls = r->sampled_out_calls;
    o->sampled_out_rows = r->sampled_out_rows;
    o->disabled_calls = r->disabled_calls;
    o->drained_bytes = r->drained_bytes;
    o->released_bytes = r->released_bytes;
    o->drain_batches = r->drain_batches;
    o->block_wait_ns = r->block_wait_ns;
    o->dev_ring_high_water = r->dev_high;
    o->host_ring_high_water = r->host_high;
    {
        std::lock_guard<std::mutex> lk(r->mu);
        uint64_t bad = 0;
        HIP_TRY(hipMemcpyAsync(&bad, &r->dctrl->bad_rows, 8, hipMemcpyDeviceToHost, r->ctl_stream));
        HIP_TRY(hipStreamSynchronize(r->ctl_stream));
        o->bad_rows = bad;
    }
    return DMI_OK;
}

dmi_status_t dmi_get_point_drops(dmi_ring_t *r, uint32_t point_id, uint64_t *n)
{
    if (!r || !n || point_id >= DMI_MAX_POINTS) return fail(DMI_ERR_INVALID_ARG, "bad argument");
    (void)hipSetDevice(r->dev);
    uint32_t v = 0;
    std::lock_guard<std::mutex> lk(r->mu);
    HIP_TRY(hipMemcpyAsync(&v, &r->dctrl->point_drops[point_id], 4, hipMemcpyDeviceToHost, r->ctl_stream));
    HIP_TRY(hipStreamSynchronize(r->ctl_stream));
    *n = v;
    return DMI_OK;
}

dmi_status_t dmi_debug_fill_rings(dmi_ring_t *r, uint8_t value)
{
    if (!r) return fail(DMI_ERR_INVALID_ARG, "ring is NULL");
    (void)hipSetDevice(r->dev);
    std::lock_guard<std::mutex> lk(r->mu);
    HIP_TRY(hipMemsetAsync(r->dev_ring, value, r->dev_cap, r->drain_stream));
    HIP_TRY(hipStreamSynchronize(r->drain_stream));
    memset(r->host_ring, value, r->host_cap);
    return DMI_OK;
}

}  // extern "C"
