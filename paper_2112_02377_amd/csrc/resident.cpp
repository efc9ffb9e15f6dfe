// Host side of the resident loop: which loops take it, its buffers, launch
// and result.
#include <algorithm>

#include "handle.h"
#include "launch.h"
#include "resident.h"

namespace jac {

namespace {

// A loop this short costs less as per-sweep launches: a cooperative launch
// takes about 20 us from queue to queue, a per-sweep launch of a small
// system 5.4 us against 1.5-2.5 us for a resident sweep.
constexpr int32_t kResMinSweeps = 8;

// The ring starts on a boundary of its own: behind 256 bytes of control words
// the 64^3 sweep took 3.2 us instead of 2.4.
constexpr size_t kResRingOff = 65536;
static_assert(sizeof(ResCtl) <= kResRingOff, "control words");

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

}  // namespace

bool run_resident(Handle& h, const SysDev& s, bool fp32, bool solve, int32_t kend, int norm_inf, double* hist,
                  const void* x0, void* xout, void* x0_out, SysState& out)
{
    const Plan& pl = h.plan;
    const int nrhs = h.nrhs;
    // Options that name a launch shape keep per-sweep launches (or the
    // persistent loop); the norm is summed in the order of 256 threads.
    if (h.opt.loop != 0 || h.opt.grid != 0 || h.opt.block != kResBlock || kend < kResMinSweeps || h.res_off)
        return false;
    const bool loc = pl.colfmt == COL_LOCAL16;
    if (!loc && pl.colfmt != COL_TABL && !(pl.colfmt == COL_TABG && !pl.res_run0.empty())) return false;
    const int per_wave = (pl.max_tile_slices + kResBlock / 64 - 1) / (kResBlock / 64);
    if (pl.ntiles < 1 || pl.max_width > kResWidth) return false;
    // rows of more entries gathered than the width's kernel holds take the next wider one
    int width = pl.max_width;
    if (pl.res_max_halo > res_halo(width) * kResBlock) width = std::max(width, 8);
    if (pl.res_max_halo > res_halo(width) * kResBlock) return false;
    const size_t ts = fp32 ? 4 : 8, vec = (size_t)h.a.n * nrhs * ts;
    if (vec >= ((size_t)1 << 32)) return false;
    void* fn = res_kernel(fp32, nrhs, width, per_wave, loc);
    if (!fn) return false;
    const int32_t ldx = pl.res_max_fp + (!loc && width > 14 ? 128 : 0);   // zeros at both ends, see resident.hip
    if ((size_t)ldx * ts > 65536) return false;          // 16-bit byte offsets
    // LDS is handed out in pieces of 1280 bytes, which the occupancy query
    // does not count; every workgroup must be resident, so round up here
    const size_t lds = (res_lds(pl, ldx, nrhs, ts, width, loc) + 1279) / 1280 * 1280;
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kResBlock, lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const int64_t grid = (int64_t)pl.ntiles + kResDeciders;
    if (grid > (int64_t)nb * num_cus()) return false;

    DeviceArrays& d = h.d;
    hipStream_t st = h.stream;
    const int npart = res_partials(nrhs, width, loc);
    const size_t o_ring = kResRingOff, o_part = o_ring + up256((size_t)kResRing * vec);
    const size_t bytes = o_part + (size_t)kResPart * pl.ntiles * npart * nrhs * sizeof(double);
    if (!d.res_work.p || d.res_work.bytes < bytes) {
        try {
            d.res_work.alloc(bytes);
        } catch (const Error& e) {
            if (e.status != JAC_E_NOMEM) throw;
            (void)hipGetLastError();
            return false;                   // per-sweep launches need none of it
        }
        launch_zero_u32(static_cast<uint32_t*>(d.res_work.p), (int32_t)(sizeof(ResCtl) / 4), st);
        h.res_next = kResPart;
        h.res_arrived = 0;
    }
    char* work = static_cast<char*>(d.res_work.p);
    ResCtl* dev = reinterpret_cast<ResCtl*>(work);
    ResSys r{};
    r.tile_row0 = s.tile_row0;
    r.tile_slice0 = s.tile_slice0;
    r.slice_off = s.slice_off;
    if (pl.colfmt == COL_TABG) {
        const int32_t* q = static_cast<const int32_t*>(d.res_plan.p);
        r.run0 = q;
        r.run_lds = q += pl.res_run0.size();
        r.run_delta = q += pl.res_run_lds.size();
        r.fp = q += pl.res_run_delta.size();
        r.own = q += pl.res_fp.size();
        r.shift = q += pl.res_own.size();
    } else {
        r.run0 = s.tile_run0;
        r.run_lds = s.run_lds;
        r.run_delta = s.run_delta;
        r.fp = s.tile_fp;
        r.own = s.tile_own;
        r.shift = s.shift;
    }
    r.col16 = s.col16;
    r.val = s.val;
    r.b = s.b;
    r.x0 = x0;
    r.xout = xout;
    r.ring = work + o_ring;
    r.part = reinterpret_cast<double*>(work + o_part);
    r.ctl = dev;
    r.n = h.a.n;
    r.ntiles = pl.ntiles;
    for (int c = 0; c < 4; ++c) {
        r.thr[c] = s.thr[c];
        r.big[c] = s.big[c];
    }
    ResParams p{};
    p.sys = r;
    p.hist = hist;
    p.kbase = h.res_next;
    p.arrive = h.res_arrived += (uint32_t)grid;
    p.nd = kResDeciders;
    p.kend = kend;
    p.solve = solve ? 1 : 0;
    p.norm_inf = norm_inf;
    if (h.opt.timing) {
        for (auto& e : h.ev)
            if (!e) JAC_HIP(hipEventCreate(&e));
        JAC_HIP(hipEventRecord(h.ev[0], st));
    }
    launch_res(fn, (int)grid, lds, ldx, st, p);
    if (h.opt.timing) JAC_HIP(hipEventRecord(h.ev[1], st));
    if (x0_out) launch_res_settle(fp32, st, xout, x0_out, (int64_t)h.a.n * nrhs, dev, p.kbase);
    ResCtl host;
    JAC_HIP(hipMemcpyAsync(&host, dev, sizeof(ResCtl), hipMemcpyDeviceToHost, st));
    h.sync();
    if (host.abort == p.kbase) {
        h.res_off = true;                   // do not wait that long again
        return false;
    }
    if (h.opt.timing) {
        float ms = 0.f;
        JAC_HIP(hipEventElapsedTime(&ms, h.ev[0], h.ev[1]));
        h.last_loop_ms = ms;
    }
    // no word of this launch lies beyond its last sweep by more than the tiles run ahead
    h.res_next = p.kbase + (uint32_t)(solve ? host.last_k : kend) + 2 * kResPart;
    h.last_grid = (int)grid;
    h.last_loop_sweeps = kend;
    for (int c = 0; c < 4; ++c) {
        out.stop_k[c] = (int32_t)(host.stop[c] - p.kbase);
        out.nrm[c] = host.nrm[c];
    }
    out.done_k = 0;
    out.status = host.status;
    out.last_k = host.last_k;
    return true;
}

}  // namespace jac
