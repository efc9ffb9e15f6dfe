// Host-only checks of what the resident sweep loop takes from its plan (no
// GPU).  Prints one summary line, or "FAIL ..." and exits 1.
//
// usage: resident_check positions N points mode nparts [sub]
//   every LDS position the loop's kernels read for an N^3 grid's matrix of
//   7-point or 27-point rows (27-point: a tenth of the edges dropped) under a
//   split (mode 1 JB, 2 JBO, 3 JSS), lanes of absent rows and slices included
//    or: resident_check layout N points mode nparts [sub]
//   the loop's footprints: every stored entry, and every clamped column that
//   a row without an entry of its slice's table reads, decodes from its LDS
//   position to the column the per-sweep launches read
//    or: resident_check numbers sweeps
//   what a solve left in the control words reads as "not yet" to every later
//   launch, over launches of that many fixed sweeps whose numbers pass 2^32,
//   and no launch has the number of the one before, new buffers between them
//   included
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "jac_internal.h"
#include "resident.h"

namespace jac {
void fail(jac_status s, const std::string& msg) { throw Error{s, msg}; }
void hip_check(hipError_t, const char*) {}
void set_last_error(const std::string&) {}
}  // namespace jac

using namespace jac;

static int bad(const char* what, long long a, long long b)
{
    printf("FAIL %s %lld %lld\n", what, a, b);
    return 1;
}

static Csr stencil(int N, int points)
{
    Csr a;
    a.n = N * N * N;
    a.rp.push_back(0);
    for (int z = 0; z < N; ++z)
        for (int y = 0; y < N; ++y)
            for (int x = 0; x < N; ++x) {
                for (int dz = -1; dz <= 1; ++dz)
                    for (int dy = -1; dy <= 1; ++dy)
                        for (int dx = -1; dx <= 1; ++dx) {
                            const int u = x + dx, v = y + dy, w = z + dz;
                            if (u < 0 || v < 0 || w < 0 || u >= N || v >= N || w >= N) continue;
                            const int far = abs(dx) + abs(dy) + abs(dz);
                            const int32_t r = x + N * (y + N * z), c = u + N * (v + N * w);
                            if (points == 7 && far > 1) continue;
                            // dropped for both rows of an edge alike
                            if (far && points == 27 && ((uint32_t)(std::min(r, c) * 2654435761u + std::max(r, c) * 40503u) >> 7) % 10 == 0)
                                continue;
                            a.ci.push_back(c);
                            a.v.push_back(far ? -1.0 : 30.0);
                        }
                a.rp.push_back((int32_t)a.ci.size());
            }
    return a;
}

static Plan plan_of(const Csr& a, int N, int mode, int P, int sg, Csr* permuted = nullptr)
{
    const int32_t grid[3] = {N, N, N}, sub[3] = {sg, sg, sg};
    Partition part = make_partition(a, mode, P, mode == JAC_SUBSTRUCT ? sub : nullptr, grid, 0);
    std::vector<int64_t> src;
    Csr pa = permute(a, part.perm, part.iperm, &src);
    PlanParams prm;
    prm.tile_rows = 512;
    prm.lds_elems = 4096;
    prm.staged = mode != JAC_BANDROW;
    prm.fill_gap = mode == JAC_BANDROW_SP ? 16 : 0;
    if (permuted) *permuted = pa;
    return make_plan(pa, part.cuts, prm);
}

static int positions(int argc, char** argv)
{
    const int N = atoi(argv[2]), points = atoi(argv[3]), mode = atoi(argv[4]), P = atoi(argv[5]);
    const Plan pl = plan_of(stencil(N, points), N, mode, P, argc > 6 ? atoi(argv[6]) : 2);
    const bool tabg = pl.colfmt == COL_TABG && !pl.res_run0.empty();
    const bool wide = pl.max_width > 14 && pl.max_width <= kResWidth && pl.colfmt != COL_LOCAL16;
    int64_t absent = 0, reads = 0;
    if (wide && (tabg || pl.colfmt == COL_TABL)) {
        const std::vector<int32_t>& shift = tabg ? pl.res_shift : pl.shift;
        const std::vector<int32_t>& fps = tabg ? pl.res_fp : pl.tile_fp;
        for (int32_t t = 0; t < pl.ntiles; ++t) {
            const int32_t r0 = pl.tile_row0[t], s0 = pl.tile_slice0[t], s1 = pl.tile_slice0[t + 1];
            for (int wave = 0; wave < kResBlock / 64; ++wave)
                for (int j = 0; j < 2; ++j) {
                    const int32_t s = s0 + wave + j * (kResBlock / 64);
                    const bool live = s < s1;
                    const int32_t w = live ? pl.slice_width[s] : 0;
                    absent += !live;
                    for (int k = 0; k < kResWidth; ++k) {
                        const int32_t tab = w > 0 ? shift[(size_t)(pl.slice_off[s] / kSlice) + std::min(k, w - 1)] : 0;
                        const int32_t sh = res_wide_shift(k, w, true, tab, r0 + (s - s0) * kSlice);
                        for (int lane = 0; lane < kSlice; ++lane, ++reads) {
                            const int32_t li = wave * 64 + lane + j * kResBlock, pos = r0 + li + sh;
                            if (pos < -2 * kResPad || pos >= fps[t] + kResPad) return bad("position", t, pos);
                            // zeros for slots past the padded width; else rows read entries that are there or copied
                            if (k >= res_padded(w, true)) {
                                if (pos >= -kResPad) return bad("zero position", t, pos);
                            } else if (r0 + li < pl.tile_row0[t + 1] &&
                                       (pos < -pl.res_under || pos >= fps[t] + pl.res_over)) {
                                return bad("row's position", t, pos);
                            }
                        }
                    }
                }
        }
        if (pl.res_under > kResPad || pl.res_over > kResPad) return bad("ends", pl.res_under, pl.res_over);
    }
    printf("wide %d ntiles %d absent %lld reads %lld\n", wide ? 1 : 0, pl.ntiles, (long long)absent, (long long)reads);
    return 0;
}

static int layout(int argc, char** argv)
{
    const int N = atoi(argv[2]), points = atoi(argv[3]), mode = atoi(argv[4]), P = atoi(argv[5]);
    const int sg = argc > 6 ? atoi(argv[6]) : 2;
    const Csr a = stencil(N, points);
    Csr pa;
    const Plan pl = plan_of(a, N, mode, P, sg, &pa);
    const bool tabg = pl.colfmt == COL_TABG && !pl.res_run0.empty(), tabl = pl.colfmt == COL_TABL;
    const bool loc = pl.colfmt == COL_LOCAL16;
    if (!tabg && !tabl && !loc) return bad("format", pl.colfmt, 0);
    const std::vector<int32_t>&run0 = tabg ? pl.res_run0 : pl.tile_run0, &run_lds = tabg ? pl.res_run_lds : pl.run_lds,
    &run_delta = tabg ? pl.res_run_delta : pl.run_delta, &fps = tabg ? pl.res_fp : pl.tile_fp,
    &own = tabg ? pl.res_own : pl.tile_own, &shift = tabg ? pl.res_shift : pl.shift;
    int64_t holes = 0, width = 0;
    for (int32_t t = 0; t < pl.ntiles; ++t) {
        const int32_t r0 = pl.tile_row0[t], r1 = pl.tile_row0[t + 1], q0 = run0[t], q1 = run0[t + 1], fp = fps[t];
        if (q1 <= q0 || run_lds[q0] != 0) return bad("runs", t, q1 - q0);
        // column of every position; ascending, inside the matrix, the own rows in one piece
        std::vector<int32_t> col((size_t)fp);
        for (int32_t e = 0, q = q0; e < fp; ++e) {
            while (q + 1 < q1 && run_lds[q + 1] <= e) ++q;
            col[e] = e + run_delta[q];
            if (col[e] < 0 || col[e] >= pa.n || (e > 0 && col[e] <= col[e - 1])) return bad("footprint", t, e);
        }
        for (int32_t i = r0; i < r1; ++i)
            if (own[t] + i - r0 >= fp || col[own[t] + i - r0] != i) return bad("own row", t, i);
        if (fp - (r1 - r0) > pl.res_max_halo || fp > pl.res_max_fp || q1 - q0 > pl.res_max_runs) return bad("maxima", t, fp);
        std::vector<char> used((size_t)fp, 0);
        for (int32_t s = pl.tile_slice0[t]; s < pl.tile_slice0[t + 1]; ++s) {
            width = std::max<int64_t>(width, pl.slice_width[s]);
            for (int32_t k = 0; k < pl.slice_width[s]; ++k)
                for (int32_t lane = 0; lane < kSlice && pl.slice_row0[s] + lane < r1; ++lane) {
                    const int32_t i = pl.slice_row0[s] + lane;
                    const int64_t g = pl.slice_off[s] / kSlice + k;
                    const int32_t pos = loc ? pl.col16[pl.slice_off[s] + (int64_t)k * kSlice + lane]
                                            : std::min(std::max(i + shift[g], 0), fp - 1);
                    if (pos >= fp) return bad("position", i, pos);
                    if (tabg && col[pos] != std::min(std::max(i + pl.shift[g], 0), pa.n - 1)) return bad("clamped", i, k);
                }
        }
        for (int32_t i = r0; i < r1; ++i)
            for (int32_t p = pa.rp[i]; p < pa.rp[i + 1]; ++p) {
                const int64_t slot = pl.slot_of_nnz[p];
                const int32_t s = pl.tile_slice0[t] + (i - r0) / kSlice;
                const int64_t k = (slot - pl.slice_off[s]) / kSlice;
                const int32_t pos = loc ? pl.col16[slot] : i + shift[pl.slice_off[s] / kSlice + k];
                if (pos < 0 || pos >= fp || col[pos] != pa.ci[p]) return bad("entry", i, p);
                used[pos] = 1;
            }
        for (int32_t e = 0; e < fp; ++e) holes += !used[e];
    }
    printf("fmt %d width %lld holes %lld ntiles %d\n", pl.colfmt, (long long)width, (long long)holes, pl.ntiles);
    return 0;
}

static int numbers(int32_t sweeps)
{
    ResNumbers nb;
    ResCtl ctl{};
    int64_t total = 0, launches = 0, clears = 0;
    uint32_t before = 0;
    for (; total < (int64_t)5 << 31; ++launches) {
        if (nb.restart()) {
            ctl = ResCtl{};
            ++clears;
        }
        if (launches == 0 || launches == 1) {
            ctl = ResCtl{};
            nb.zeroed();
        }
        const uint32_t kbase = nb.next;
        if (kbase == before) return bad("number used again", total, kbase);
        before = kbase;
        for (int d = 0; d < kResDeciders; ++d)
            if ((int32_t)(ctl.word[d] - kbase) >= 0) return bad("word", total, ctl.word[d]);
        for (uint32_t w : ctl.stop)
            if ((int32_t)(w - kbase) >= 0) return bad("stop word", total, w);
        if (ctl.done == kbase || ctl.abort == kbase) return bad("done or abort", total, kbase);
        const bool solve = launches == 2;
        const int32_t last = solve ? 5 : sweeps;
        // the deciding workgroups' last words; stop words and done by solves alone
        for (int d = 0; d < kResDeciders; ++d) ctl.word[d] = kbase + (uint32_t)last + kResDeciders - 1;
        if (solve)
            for (uint32_t& w : ctl.stop) w = kbase + 5;
        if (solve) ctl.done = kbase;
        nb.passed(last);
        total += last;
    }
    printf("launches %lld clears %lld\n", (long long)launches, (long long)clears);
    return 0;
}

int main(int argc, char** argv)
{
    try {
        if (argc == 3 && !strcmp(argv[1], "numbers")) return numbers(atoi(argv[2]));
        if (argc >= 6 && !strcmp(argv[1], "positions")) return positions(argc, argv);
        if (argc >= 6 && !strcmp(argv[1], "layout")) return layout(argc, argv);
    } catch (Error& e) {
        printf("FAIL error %d %s\n", (int)e.status, e.msg.c_str());
        return 1;
    }
    return 2;
}
