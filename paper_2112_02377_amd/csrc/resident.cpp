// Host side of the resident loop: which loops take it, its buffers, launch
// and result.
#include <algorithm>
#include <chrono>
#include <limits>
#include <mutex>
#include <thread>

#include "handle.h"
#include "launch.h"
#include "resident.h"

namespace jac {

namespace {

// A shorter loop costs less as per-sweep launches: a resident launch clears
// its ring and loads its matrix first.  Eight sweeps, launched per sweep and
// resident: 16^3 73 and 36 us, 64^3 87 and 79, 56^3 of 27-point rows 138 and
// 89.  With rows of a 7-point matrix, beyond some 640 tiles or 4 MB of x the
// start takes longer than eight sweeps gain: 72^3 97 and 108 us at eight, 152
// and 138 at sixteen; 80^3 118 and 141, 196 and 179; 84^3 129 and 169, 216 and
// 216; 64^3 of four columns 137 and 148, 229 and 217 (48^3 of four: 100 and 73).
constexpr int32_t kResMinSweeps = 8, kResMinSweepsLarge = 16;
constexpr int32_t kResLargeTiles = 640;
constexpr size_t kResLargeBytes = 4000000;
// Sweeps of one launch at most: it occupies its compute units until it ends
// (65536 sweeps are 0.15 to 0.35 s), where other streams' work got its turn
// between per-sweep launches.  Longer loops are several launches; one more
// costs about 20 us.
constexpr int32_t kResMaxSweeps = 1 << 16;

// The ring starts on a boundary of its own, clear of the control words (its
// distance from them made no difference: 64 KiB, 320 KiB and 2 MiB measured).
constexpr size_t kResRingOff = 65536;
static_assert(sizeof(ResCtl) <= kResRingOff, "control words");

// Launches of a loop, of about equal length (none of several below half the most).
int32_t res_launches(int32_t sweeps) { return (int32_t)(((int64_t)sweeps + kResMaxSweeps - 1) / kResMaxSweeps); }

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

// LDS of a workgroup: x of the footprint, once or twice (or, before the loop,
// the runs), control words; for wide rows the gather offsets and either
// explicit positions or b of two slices per wave.
size_t res_lds(const Plan& pl, int32_t ldx, int nrhs, size_t elem, int width, bool loc)
{
    const size_t x = (res_two_buffers(nrhs, width, loc) ? 2 : 1) * res_x_bytes(ldx, nrhs, elem);
    size_t b = kResCtlWords * 4;
    if (width > 14) b += (size_t)res_halo(width) * kResBlock * 4;
    if (width > 14 && loc) b += (size_t)((kResWidth + 3) / 4) * 2 * kResBlock * 8;
    if (res_rhs_in_lds(elem, nrhs, width, loc)) b += 2 * kResBlock * elem;
    const size_t decider = kResRed * 8 + 32;
    return std::max({x + b, (size_t)pl.res_max_runs * 8, decider});
}

// Resident launches on a device that may not have ended, one entry per stream
// (a stream runs one at a time).  Workgroups of a launch wait for each other,
// so two launches may be on the device together only if both fit whole: a
// launch joins others if their shares of the device and the largest workgroup's
// share of a compute unit make no more than 1 -- then some compute unit always
// has room for the next workgroup, whatever the order.
struct Loop {
    const Handle* holder;
    hipStream_t stream;
    const ResSeen* seen;            // of the holder
    uint32_t kbase;                 // its last launch
    double share, wg;
};
// A call that waits for room, in the order in which they came.
using Clock = std::chrono::steady_clock;
struct Waiter {
    const Handle* h;
    Clock::time_point since;
};
constexpr int kMaxDevices = 64;
std::mutex g_loops_mutex;
std::vector<Loop> g_loops[kMaxDevices];
std::vector<Waiter> g_waiters[kMaxDevices];
// Nobody enters past a call that has waited this long: without that a thread
// with one loop after the other kept another out for 100 ms (two threads with
// 4 ms solves at 64^3); with it the longest call takes 8.5.
constexpr auto kPatience = std::chrono::milliseconds(2);

// Whether a launch of that share may go on the handle's stream.  Waits for
// room, but only behind launches that are running: one behind other work on
// its stream may take any time.  (Per-sweep launches beside a resident loop
// that fills the device slow both: eight streams' sweeps at 64^3 take 745 us
// a hundred so, 370 one loop after the other.)
enum class Entry { no, beside, alone };
Entry loops_enter(const Handle& h, double share, double wg)
{
    if (h.device < 0 || h.device >= kMaxDevices) return Entry::no;
    int held = 0;
    std::vector<Waiter>& waiters = g_waiters[h.device];
    auto mine = [&](const Waiter& w) { return w.h == &h; };
    auto leave = [&]() { waiters.erase(std::remove_if(waiters.begin(), waiters.end(), mine), waiters.end()); };
    for (int tries = 0; tries < 20000; ++tries) {
        {
            std::lock_guard<std::mutex> lock(g_loops_mutex);
            std::vector<Loop>& v = g_loops[h.device];
            const Clock::time_point now = Clock::now();
            const bool after = !waiters.empty() && waiters.front().h != &h && now - waiters.front().since > kPatience;
            Loop me{&h, h.stream, static_cast<const ResSeen*>(h.d.res_seen.p), h.res_numbers.next, share, wg};
            double total = 0.0, most = wg;
            bool running = true;
            for (auto q = v.begin(); q != v.end();) {
                if (__atomic_load_n(&q->seen->ended, __ATOMIC_ACQUIRE) == q->kbase) {
                    q = v.erase(q);
                } else if (q->holder == &h || (q->stream == h.stream && h.stream != hipStreamPerThread)) {
                    me.share = std::max(me.share, q->share);
                    me.wg = std::max(me.wg, q->wg);
                    ++q;
                } else {
                    total += q->share;
                    most = std::max(most, q->wg);
                    running = running && __atomic_load_n(&q->seen->started, __ATOMIC_RELAXED) == q->kbase;
                    ++q;
                }
            }
            const bool fits = total == 0.0 || total + me.share + std::max(most, me.wg) <= 1.0;
            if (fits && !after) {
                leave();
                v.erase(std::remove_if(v.begin(), v.end(),
                                       [&](const Loop& q) {
                                           return q.holder == &h ||
                                                  (q.stream == h.stream && h.stream != hipStreamPerThread);
                                       }),
                        v.end());
                v.push_back(me);
                return total == 0.0 ? Entry::alone : Entry::beside;
            }
            held = running ? 0 : held + 1;       // a launch takes some time to start, too
            if (held > 10) {
                leave();
                return Entry::no;
            }
            if (std::none_of(waiters.begin(), waiters.end(), mine)) waiters.push_back({&h, now});
        }
        std::this_thread::sleep_for(std::chrono::microseconds(20));
    }
    std::lock_guard<std::mutex> lock(g_loops_mutex);
    leave();
    return Entry::no;
}

// Ordinary launches, since cooperative ones run one after another, behind any
// that its stream holds back, and one process at a time: four threads with
// solves at 20^3 take 0.50 ms a solve, 1.8 as cooperative launches (1.27 per
// sweep); 33^3 1.4, 4.1 and 3.0; 64^3, of which two do not fit, 20.7, 22.9
// and 32.  A call of ten sweeps at 16^3 takes 81 us, 101 cooperative.  But
// sweeps are about 1% slower (2216 at 65^3: 12.25 and 12.12 ms, 1160 at 20^3:
// 2.84 and 2.81; cause not found), so a launch that may be long is
// cooperative where no other stream's is on the device.
constexpr int32_t kResLong = 1024;

// What a launch needs besides its system; ok: the plan fits the chip and the
// handle's options leave the choice open.
struct ResLaunch {
    bool ok = false;
    void* fn = nullptr;
    int grid = 0;
    size_t lds = 0;
    int32_t ldx = 0;
    double share = 0.0, wg = 0.0;   // of the device, and a workgroup's of a compute unit
    size_t bytes = 0, o_part = 0;   // of the handle's buffer; where the partials start
    bool loc = false, tabg = false, wide = false;
    ResParams p{};
};

// Whether the loop takes the plan, and how (nothing is allocated).
ResLaunch res_shape(const Handle& h, const Plan& pl, bool fp32, int nrhs, int32_t kend, bool adjoint)
{
    ResLaunch L;
    // Options that name a launch shape keep per-sweep launches (or the
    // persistent loop); the norm is summed in the order of 256 threads.
    if (h.opt.loop != 0 || (h.opt.grid != 0 && !h.res_tuned) || h.opt.block != kResBlock) return L;
    if (kend < kResMinSweeps || kend > kResMaxSweeps) return L;
    const bool loc = pl.colfmt == COL_LOCAL16;
    const bool tabg = pl.colfmt == COL_TABG && !pl.res_run0.empty();
    if (!tabg && (adjoint || (!loc && pl.colfmt != COL_TABL))) return L;
    const int per_wave = (pl.max_tile_slices + kResBlock / 64 - 1) / (kResBlock / 64);
    if (pl.ntiles < 1 || pl.max_width > kResWidth) return L;
    // rows of more entries gathered than the width's kernel holds take the next wider one
    int width = pl.max_width;
    if (pl.res_max_halo > res_halo(width) * kResBlock) width = std::max(width, 8);
    const bool wide = width > 14 && !loc;
    const int32_t ends = wide ? pl.res_under + pl.res_over : 0;      // gathered with the entries of other tiles
    if (pl.res_max_halo + ends > res_halo(width) * kResBlock) return L;
    const size_t ts = fp32 ? 4 : 8, vec = (size_t)h.a.n * nrhs * ts;
    if (vec >= ((size_t)1 << 32)) return L;              // 32-bit byte offsets into a ring slot
    if (width <= 14 && (pl.ntiles > kResLargeTiles || vec > kResLargeBytes) && kend < kResMinSweepsLarge) return L;
    L.fn = adjoint ? res_adjoint_kernel(width, per_wave) : res_kernel(fp32, nrhs, width, per_wave, loc);
    if (!L.fn) return L;
    L.ldx = pl.res_max_fp + (wide ? kResEnds : 1);       // and a zero for slots past a slice's width
    if ((size_t)L.ldx * ts > 65536) return L;            // 16-bit byte offsets
    // LDS is handed out in pieces of 1280 bytes, which the occupancy query
    // does not count; every workgroup must be resident, so round up here
    L.lds = (res_lds(pl, L.ldx, nrhs, ts, width, loc) + 1279) / 1280 * 1280;
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, L.fn, kResBlock, L.lds) != hipSuccess) {
        (void)hipGetLastError();
        return L;
    }
    L.grid = pl.ntiles + kResDeciders;
    if (L.grid > (int64_t)nb * num_cus()) return L;
    // the dispatcher deals workgroups to groups of eight compute units in turn
    const int groups = std::max(num_cus() / 8, 1);
    L.share = (double)((L.grid + groups - 1) / groups) / (8.0 * nb);
    L.wg = 1.0 / nb;
    L.o_part = kResRingOff + up256((size_t)kResRing * vec);
    L.bytes = L.o_part + (size_t)kResPart * pl.ntiles * res_partials(nrhs, width, loc) * nrhs * sizeof(double);
    L.loc = loc;
    L.tabg = tabg;
    L.wide = wide;
    L.ok = true;
    return L;
}

ResLaunch res_prepare(Handle& h, const Plan& pl, const DeviceArrays& pd, bool fp32, int nrhs, int32_t kend, bool adjoint)
{
    h.res_poll();
    ResLaunch L = res_shape(h, pl, fp32, nrhs, kend, adjoint);
    if (!L.ok) return L;
    L.ok = false;
    // A captured launch would carry the numbers of this one at every replay.
    // (The per-sweep loop cannot be captured either: it waits for its stream.)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h.stream, &capture) != hipSuccess) (void)hipGetLastError();
    else if (capture != hipStreamCaptureStatusNone)
        fail(JAC_E_HIP, "the stream is being captured; of the sweep loops only jac_sweep_noalloc can be");
    if (!h.res_retry.now()) return L;
    DeviceArrays& d = h.d;
    const bool tabg = L.tabg, wide = L.wide;
    bool clear = h.res_numbers.restart();
    if (!d.res_work.p || d.res_work.bytes < L.bytes) {
        try {
            d.res_work.alloc(L.bytes);
        } catch (const Error& e) {
            if (e.status != JAC_E_NOMEM) throw;
            (void)hipGetLastError();
            return L;                       // per-sweep launches need none of it
        }
        h.res_numbers.zeroed();
        clear = true;
    }
    if (clear) launch_zero_u32(static_cast<uint32_t*>(d.res_work.p), (int32_t)(sizeof(ResCtl) / 4), h.stream);
    char* work = static_cast<char*>(d.res_work.p);
    ResSys& r = L.p.sys;
    r.tile_row0 = static_cast<const int32_t*>(pd.tile_row0.p);
    r.tile_slice0 = static_cast<const int32_t*>(pd.tile_slice0.p);
    r.slice_off = static_cast<const int64_t*>(pd.slice_off.p);
    if (tabg) {
        const int32_t* q = static_cast<const int32_t*>(pd.res_plan.p);
        r.run0 = q;
        r.run_lds = q += pl.res_run0.size();
        r.run_delta = q += pl.res_run_lds.size();
        r.fp = q += pl.res_run_delta.size();
        r.own = q += pl.res_fp.size();
        r.shift = q += pl.res_own.size();
    } else {
        r.run0 = static_cast<const int32_t*>(pd.tile_run0.p);
        r.run_lds = static_cast<const int32_t*>(pd.run_lds.p);
        r.run_delta = static_cast<const int32_t*>(pd.run_delta.p);
        r.fp = static_cast<const int32_t*>(pd.tile_fp.p);
        r.own = static_cast<const int32_t*>(pd.tile_own.p);
        r.shift = static_cast<const int32_t*>(pd.shift.p);
    }
    r.col16 = static_cast<const uint16_t*>(pd.col16.p);
    r.ring = work + kResRingOff;
    r.part = reinterpret_cast<double*>(work + L.o_part);
    r.ctl = reinterpret_cast<ResCtl*>(work);
    r.n = h.a.n;
    r.ntiles = pl.ntiles;
    r.under = wide ? pl.res_under : 0;
    r.over = wide ? pl.res_over : 0;
    L.p.kend = kend;
    L.p.wait = h.opt.loop_wait_us * 100;
    L.p.nd = kResDeciders;
    L.ok = true;
    return L;
}

// Puts it on the stream; false if other streams' loops leave it no room, or
// (and not tried again for a while) if it was refused.
bool res_launch(Handle& h, ResLaunch& L)
{
    const Entry entry = loops_enter(h, L.share, L.wg);
    if (entry == Entry::no) return false;
    L.p.seen = static_cast<ResSeen*>(h.d.res_seen.p);
    L.p.kbase = h.res_numbers.next;
    L.p.arrive = h.res_numbers.arrived + (uint32_t)L.grid;
    if (h.opt.timing) {
        for (auto& e : h.ev)
            if (!e) JAC_HIP(hipEventCreate(&e));
        JAC_HIP(hipEventRecord(h.ev[0], h.stream));
    }
    bool launched = false;
    if (entry == Entry::alone && L.p.solve && L.p.kend > kResLong && !h.res_ordinary) {
        launched = launch_res(L.fn, L.grid, L.lds, L.ldx, h.stream, L.p, true) == hipSuccess;
        if (!launched) {
            (void)hipGetLastError();
            h.res_ordinary = true;          // refused while another process has cooperative launches
        }
    }
    if (!launched && launch_res(L.fn, L.grid, L.lds, L.ldx, h.stream, L.p, false) != hipSuccess) {
        (void)hipGetLastError();
        h.res_leave();
        h.res_retry.failed();
        return false;
    }
    h.res_numbers.arrived = L.p.arrive;
    if (h.opt.timing) JAC_HIP(hipEventRecord(h.ev[1], h.stream));
    return true;
}

void res_time(Handle& h)
{
    if (!h.opt.timing) return;
    JAC_HIP(hipEventSynchronize(h.ev[1]));
    float ms = 0.f;
    JAC_HIP(hipEventElapsedTime(&ms, h.ev[0], h.ev[1]));
    h.last_loop_ms = ms;
}

// Waits for a launch and reads its result; false if it gave up.
bool res_wait(Handle& h, const ResLaunch& L, ResCtl& host)
{
    JAC_HIP(hipMemcpyAsync(&host, L.p.sys.ctl, sizeof(ResCtl), hipMemcpyDeviceToHost, h.stream));
    h.sync();
    h.res_leave();
    if (host.abort == L.p.kbase) {
        h.res_numbers.passed(L.p.kend);
        h.res_retry.failed();               // do not wait that long again soon
        return false;
    }
    h.res_retry.ran();
    ++h.res_loops;
    res_time(h);
    h.res_numbers.passed(L.p.solve ? host.last_k : L.p.kend);
    return true;
}

}  // namespace

void Handle::res_leave()
{
    if (device < 0 || device >= kMaxDevices) return;
    std::lock_guard<std::mutex> lock(g_loops_mutex);
    std::vector<Loop>& v = g_loops[device];
    v.erase(std::remove_if(v.begin(), v.end(), [&](const Loop& q) { return q.holder == this; }), v.end());
}

void Handle::res_poll()
{
    const ResSeen* s = static_cast<const ResSeen*>(d.res_seen.p);
    const uint32_t ended = __atomic_load_n(&s->ended, __ATOMIC_ACQUIRE);
    const uint32_t failed = __atomic_load_n(&s->gave_up, __ATOMIC_RELAXED) - res_gave_up;
    if (failed) {
        res_gave_up += failed;
        res_loops -= (int32_t)failed;
        res_retry.failed();
    } else if (res_open && ended == res_open) {
        res_retry.ran();
        res_open = 0;
    }
}

// Fixed FP64 sweeps of one launch, x_0 in x0 (null: zero), x_K to x0_out.
static bool res_sweeps(Handle& h, const SysDev& s, int32_t kend, double* hist, const void* x0, void* xout, void* x0_out,
                       double* xall)
{
    ResLaunch L = res_prepare(h, h.plan, h.d, false, h.nrhs, kend, false);
    if (!L.ok) return false;
    ResSys& r = L.p.sys;
    r.val = s.val;
    r.b = s.b;
    r.x0 = x0;
    r.xout = xout;
    L.p.hist = hist;
    L.p.xall = xall;
    if (!res_launch(h, L)) return false;
    launch_res_finish(h.nrhs, L.loc, h.plan.res_max_runs, h.stream, L.p,
                      static_cast<double*>(x0_out));
    h.res_numbers.passed(kend);
    h.res_open = L.p.kbase;
    ++h.res_loops;
    res_time(h);
    h.last_grid = L.grid;
    return true;
}

int32_t run_resident_sweeps(Handle& h, const SysDev& s, int32_t K, double* hist, const void* x0, void* xout, void* x0_out,
                            double* xall)
{
    const int32_t launches = res_launches(K);
    double ms = 0.0;
    int32_t done = 0;
    for (int32_t q = 0; q < launches; ++q) {
        const int32_t k1 = (int32_t)((int64_t)K * (q + 1) / launches);
        if (!res_sweeps(h, s, k1 - done, hist ? hist + (int64_t)done * h.nrhs : nullptr, q == 0 ? x0 : x0_out, xout,
                        x0_out, xall ? xall + (int64_t)done * h.a.n : nullptr))
            break;
        done = k1;
        ms += h.last_loop_ms;
    }
    if (done) {
        h.last_loop_sweeps = done;
        if (h.opt.timing) h.last_loop_ms = ms;
    }
    return done;
}

// One launch of a solve; false also when it gave up.  x0_out (null: not
// wanted) receives the iterate, unless more sweeps follow and a column needs them.
static bool res_solve(Handle& h, const SysDev& s, bool fp32, int32_t kend, int norm_inf, const void* x0, void* xout,
                      void* x0_out, bool more, SysState& out)
{
    ResLaunch L = res_prepare(h, h.plan, h.d, fp32, h.nrhs, kend, false);
    if (!L.ok) return false;
    ResSys& r = L.p.sys;
    r.val = s.val;
    r.b = s.b;
    r.x0 = x0;
    r.xout = xout;
    for (int c = 0; c < 4; ++c) {
        r.thr[c] = s.thr[c];
        r.big[c] = s.big[c];
    }
    L.p.solve = 1;
    L.p.norm_inf = norm_inf;
    if (!res_launch(h, L)) return false;
    if (x0_out)
        launch_res_settle(fp32, h.stream, xout, x0_out, (int64_t)h.a.n * h.nrhs, r.ctl, L.p.kbase, more);
    ResCtl host;
    if (!res_wait(h, L, host)) return false;
    h.last_grid = L.grid;
    for (int c = 0; c < 4; ++c) {
        out.stop_k[c] = (int32_t)(host.stop[c] - L.p.kbase);
        out.nrm[c] = host.nrm[c];
    }
    out.done_k = 0;
    out.status = host.status;
    out.last_k = host.last_k;
    return true;
}

bool run_resident_solve(Handle& h, const SysDev& s, bool fp32, int32_t maxit, int norm_inf, const void* x0, void* x0_out,
                        void* xa, void* xb, SysState& out)
{
    // Each launch goes on from where the one before ran out of sweeps and
    // tests that iterate again, with the same result; a column that has
    // stopped stops at once.
    const int32_t launches = std::max(res_launches(maxit), 1);
    const bool direct = launches == 1 && x0 != x0_out;
    SysDev t = s;
    const void* from = x0;
    void* to = direct ? x0_out : xa;
    int32_t done = 0;
    uint32_t stopped = 0;
    double ms = 0.0;
    for (int32_t q = 0; q < launches; ++q) {
        const int32_t k1 = (int32_t)((int64_t)maxit * (q + 1) / launches);
        const bool more = q + 1 < launches;
        SysState st;
        if (!res_solve(h, t, fp32, k1 - done, norm_inf, from, to, direct ? nullptr : x0_out, more, st)) return false;
        ms += h.last_loop_ms;
        out.done_k = 0;
        out.status = st.status;
        out.last_k = done + st.last_k;
        const bool goes_on = more && st.status == JAC_NOT_CONVERGED;
        for (int c = 0; c < 4; ++c) {
            if ((stopped >> c) & 1u) continue;
            out.stop_k[c] = done + st.stop_k[c];
            out.nrm[c] = st.nrm[c];
            if (c < h.nrhs && goes_on && st.nrm[c] <= s.thr[c]) {
                stopped |= 1u << c;
                t.thr[c] = std::numeric_limits<double>::infinity();
            }
        }
        if (!goes_on) break;
        done = k1;
        from = to;
        to = to == xa ? xb : xa;
    }
    if (h.opt.timing) h.last_loop_ms = ms;
    return true;
}

size_t resident_adjoint_bytes(const Handle& h, int32_t K)
{
    const ResLaunch L = res_shape(h, h.tplan, false, 1, K - 1, true);
    return L.ok ? (size_t)K * h.a.n * sizeof(double) + L.bytes : 0;
}

bool run_resident_adjoint(Handle& h, int32_t K, const double* lam, double* mu, double* gb)
{
    ResLaunch L = res_prepare(h, h.tplan, h.td, false, 1, K - 1, true);
    if (!L.ok) return false;
    ResSys& r = L.p.sys;
    r.val = h.td.val.p;
    r.b = lam;
    r.invd = h.d.invd.p;
    r.xout = gb;
    L.p.xall = mu;
    ResCtl host;
    const double ms = h.last_loop_ms;
    const bool ok = res_launch(h, L) && res_wait(h, L, host);
    h.last_loop_ms = ms;                    // the forward's
    return ok;
}

}  // namespace jac
