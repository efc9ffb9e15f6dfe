// Resident sweep loop of libjacobi for gfx950: every sweep of a system in one
// launch, with the matrix held in registers.
//
// A system whose tiles all fit the chip at once (the 128 MB of vector
// registers hold the slot values) is swept without a launch per sweep and
// without reading the matrix again: workgroup t owns tile t for the whole
// loop, each lane the slots of its rows.  Per sweep a tile only gathers the
// x entries its footprint shares with other tiles, and publishes its own.
// What bounds a sweep is then the trip of a value from one workgroup to
// another through device-coherent memory (about 1.0-1.5 us measured with up
// to 256 workgroups, 1.8 us with 512), where a launch per sweep costs
// 4.8 us at 20^3 and 5.8 us at 64^3.  A sweep of this loop takes 1.9 us in
// fixed sweeps and 2.2 in solves at 20^3, 3.2 at 64^3, and with 27 slots a
// row 3.1 at 33^3, 4.4 at 56^3, 5.4 at 65^3.  Whole solves, a launch per sweep
// against this loop: 20^3 Laplacian 7.10 and 2.81 ms, 33^3 and 65^3 Q1 cubes
// 6.54 and 2.39, 39.2 and 12.1 ms, 56^3 27-point matrix 4.87 and 1.67 ms.
//
// Exchange without fences or barriers across workgroups: x_k is published in
// slot k mod 8 of a ring with relaxed device-scope stores, one per value.  A
// slot not yet written holds a sentinel (a NaN pattern the kernel never
// publishes), so a value validates itself: the reader repeats its load until
// the sentinel is gone.  The owner puts the sentinel back into the slot of
// sweep k+3 during sweep k, and waits for that store before it publishes
// x_{k+2}; a reader that asks for x_{k+3} has read the owner's x_{k+2}, so it
// cannot meet the old value.
//
// Norm and stop test: waves store their partials (summed in the order of the
// per-sweep launches, so norms are bit-identical) in a ring of sentinel
// words; deciding workgroups collect a sweep's partials, decide, and publish
// the last sweep they decided.  A tile overwrites the slot of x_j only after
// sweep j is decided: every tile has then gathered x_j, and if x_j passed the
// test its owner has copied it out.  So the tiles run ahead of the decisions
// by up to five sweeps and no wait for a decision is on the critical path.
//
// A launch starts by clearing the ring itself (every access to the shared
// words is device-coherent, none relies on what a kernel boundary does to the
// caches) and waits once for all workgroups to have done so.
//
// Every wait is bounded by the clock (2 s unless JAC_OPT_LOOP_WAIT says
// otherwise); when one runs out all workgroups leave and the loop is done
// again: a solve or the adjoint by the host, with a launch per sweep; fixed
// sweeps, which the host does not wait for, by the kernel that would have
// copied their result.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "device.h"
#include "jac_internal.h"
#include "resident.h"

namespace jac {

namespace {

constexpr int32_t kNever = kRunning;
// Longest wait for all workgroups of a launch to be there, 0.2 s: they are as
// soon as other kernels on the device leave room, unless another process's
// resident launch and this one each keep what the other needs.
constexpr uint32_t kArriveTicks = 20000000;

template <typename T> struct Bits;
template <> struct Bits<double> {
    using type = uint64_t;
    static constexpr type sentinel = 0x7ff8a5c3deadf00dull;
};
template <> struct Bits<float> {
    using type = uint32_t;
    static constexpr type sentinel = 0x7fc5a3adu;
};

template <typename V>
__device__ __forceinline__ V ldc(const V* p)
{
    return __hip_atomic_load((gptr<const V>)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ void stc(V* p, V v)
{
    __hip_atomic_store((gptr<V>)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The same at a 32-bit byte offset from a uniform base (the host bounds a
// ring slot below 4 GiB): one offset register instead of a 64-bit address.
// (The empty asm keeps the compiler from widening the offset ahead of the
// loop, which holds a register pair per access.)
template <typename V>
__device__ __forceinline__ V ldo(const V* base, uint32_t off)
{
    asm volatile("" : "+v"(off));
    return __hip_atomic_load((gptr<const V>)((gptr<const char>)base + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ void sto(V* base, uint32_t off, V v)
{
    asm volatile("" : "+v"(off));
    __hip_atomic_store((gptr<V>)((gptr<char>)base + off), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wait for this wave's own memory operations.
__device__ __forceinline__ void wait_own()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
// Workgroup barrier that orders LDS only: global loads and stores stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A bounded wait: true once it has run out or another workgroup gave up.
// (Kernel arguments, read where they are needed; no wait at all: the first
// value that is not there yet ends the launch.)
struct Patience {
    uint64_t t0 = 0;
    uint32_t n = 0;
    __device__ __forceinline__ bool out(const ResParams& P, uint32_t most = ~0u)
    {
        ResCtl* ctl = P.sys.ctl;
        const uint32_t kbase = P.kbase;
        if ((++n & 63u) != 0 && P.wait != 0) return false;
        const uint64_t t = wall_clock64();
        if (t0 == 0) t0 = t;
        if (ldc(&ctl->abort) == kbase) return true;
        if (P.wait == 0 || t - t0 > min(P.wait, most)) {
            stc(&ctl->abort, kbase);
            return true;
        }
        return false;
    }
};

// Waits until every workgroup of the launch has cleared its share of the
// ring; false if the wait ran out.
__device__ __forceinline__ bool res_arrive(const ResParams& P, int32_t* ok)
{
    ResCtl* ctl = P.sys.ctl;
    wait_own();                                     // this thread's stores have reached the device
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(&ctl->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        Patience wait;
        bool in = true;
        while ((int32_t)(ldc(&ctl->arrived) - P.arrive) < 0)
            if (wait.out(P, kArriveTicks)) {
                in = false;
                break;
            }
        *ok = in ? 1 : 0;
    }
    __syncthreads();
    return *ok != 0;
}

// The deciding workgroup d of a system: sweeps d, d + nd, ...
// NW: partials per tile and column (one per wave, or one).
template <int NRHS, int NW>
__device__ void res_decide(const ResParams& P, int32_t d, double* red)
{
    const ResSys& S = P.sys;
    const uint32_t kbase = P.kbase;
    using B = Bits<double>;
    ResCtl* ctl = S.ctl;
    const bool is_max = P.norm_inf != 0;
    constexpr int NP = NW * NRHS;
    const int32_t m = S.ntiles * NP;
    uint32_t stopped = 0;                           // columns known to have stopped
    int32_t* flag = reinterpret_cast<int32_t*>(red + kResRed);
    const int32_t klast = P.solve ? P.kend : P.kend - 1;
    for (int32_t k = d; k <= klast; k += P.nd) {
        uint64_t* part = reinterpret_cast<uint64_t*>(S.part) + (int64_t)(k % kResPart) * m;
        double v[NRHS];
#pragma unroll
        for (int c = 0; c < NRHS; ++c) v[c] = 0.0;
        bool leave = false;
        Patience wait;
        // several tiles' partials are asked for together
        constexpr int G = 4;
        for (int32_t t0 = threadIdx.x; t0 < S.ntiles && !leave; t0 += G * kResBlock) {
            uint64_t w[G][NP];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const uint64_t* from = part + (int64_t)min(t0 + g * kResBlock, S.ntiles - 1) * NP;
#pragma unroll
                for (int q = 0; q < NP; ++q) w[g][q] = ldc(&from[q]);
            }
            for (;;) {
                bool miss = false;
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int q = 0; q < NP; ++q) miss |= w[g][q] == B::sentinel && t0 + g * kResBlock < S.ntiles;
                if (!miss) break;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint64_t* from = part + (int64_t)min(t0 + g * kResBlock, S.ntiles - 1) * NP;
#pragma unroll
                    for (int q = 0; q < NP; ++q)
                        if (w[g][q] == B::sentinel) w[g][q] = ldc(&from[q]);
                }
                if (wait.out(P) || ((wait.n & 7u) == 0 && ldc(&ctl->done) == kbase)) {
                    leave = true;
                    break;
                }
            }
            // the waves' partials in order, then the tiles'
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int32_t t = t0 + g * kResBlock;
                if (t >= S.ntiles) break;
#pragma unroll
                for (int c = 0; c < NRHS; ++c) {
                    double p = __longlong_as_double((long long)w[g][c]);
#pragma unroll
                    for (int q = 1; q < NW; ++q) {
                        const double o = __longlong_as_double((long long)w[g][q * NRHS + c]);
                        p = is_max ? maxnan(p, o) : p + o;
                    }
                    v[c] = is_max ? maxnan(v[c], p) : v[c] + p;
                }
                if (!leave) {
#pragma unroll
                    for (int q = 0; q < NP; ++q) stc(&part[(int64_t)t * NP + q], (uint64_t)B::sentinel);
                }
            }
        }
        wait_own();                                 // the partials are cleared before the sweep counts as decided
        if (threadIdx.x == 0) *flag = 0;
        __syncthreads();
        if (leave) *flag = 1;
        block_reduce<NRHS>(v, is_max, red);
        const bool gone = *flag != 0;
        __syncthreads();                            // flag is written again below
        if (gone) return;
        if (threadIdx.x == 0) {
            bool event = false;
            double nrm[NRHS];
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                nrm[c] = is_max ? v[c] : sqrt(v[c]);
                if (P.hist) P.hist[(int64_t)k * NRHS + c] = nrm[c];
                if (P.solve && !((stopped >> c) & 1u) && (!(nrm[c] <= S.big[c]) || nrm[c] <= S.thr[c] || k >= P.kend))
                    event = true;
            }
            if (event) {
                // earlier sweeps decide first -- unless one of them has stopped
                // the last column, after which the others may have left
                Patience w2;
                bool over = false;
                for (int32_t j = max(0, k - P.nd + 1); j < k && !over; ++j)
                    while ((int32_t)(ldc(&ctl->word[j & (P.nd - 1)]) - kbase) < j) {
                        over = ldc(&ctl->done) == kbase || w2.out(P);
                        if (over) break;
                    }
                if (over) stopped = (1u << NRHS) - 1u;
                else {
                    asm volatile("" ::: "memory");
                    int32_t st[NRHS];
                    bool diverged = false, exhausted = false, running = false;
#pragma unroll
                    for (int c = 0; c < NRHS; ++c) {
                        st[c] = (int32_t)(ldc(&ctl->stop[c]) - kbase);
                        if (st[c] >= 0) continue;
                        st[c] = kNever;
                        stc(&ctl->nrm[c], nrm[c]);
                        if (!(nrm[c] <= S.big[c])) diverged = true;
                        else if (nrm[c] <= S.thr[c]) st[c] = k;
                        else if (k >= P.kend) { st[c] = k; exhausted = true; }
                        else running = true;
                    }
                    if (diverged) {
#pragma unroll
                        for (int c = 0; c < NRHS; ++c)
                            if (st[c] >= k) st[c] = k;
                        running = false;
                        stc(&ctl->status, (int32_t)JAC_E_DIVERGED);
                    } else if (exhausted && ldc(&ctl->status) == JAC_OK) {
                        stc(&ctl->status, (int32_t)JAC_NOT_CONVERGED);
                    }
#pragma unroll
                    for (int c = 0; c < NRHS; ++c) {
                        if (st[c] == kNever) continue;
                        if (st[c] == k) stc(&ctl->last_k, k);
                        stc(&ctl->stop[c], kbase + (uint32_t)st[c]);
                        stopped |= 1u << c;
                    }
                    wait_own();
                    if (!running) stc(&ctl->done, kbase);
                }
            }
            wait_own();
            stc(&ctl->word[d], kbase + (uint32_t)k);
            *flag = stopped;
        }
        __syncthreads();
        stopped = (uint32_t)*flag;
        if (stopped == (1u << NRHS) - 1u) return;
        __syncthreads();
    }
}

// One tile for the whole loop.  W: slots per row held, SPL: slices per wave,
// LOC: explicit LDS position per slot (else from the slice's shift table).
//
// A slot's LDS position is kept as a 16-bit byte offset, two per register
// (one vector instruction to unpack).  For W > 14 that would cost a wave per
// SIMD, and with it tiles that fit the chip: there explicit positions sit in
// LDS, four per 8 bytes, and a shift table takes one register per slice,
// lane k holding slot k's shift (a lane read and an addition per slot; rows
// without an entry of the shift reach at most 63 entries past either end of
// the footprint, where copies of its first and last entry are kept).  Both slices of a wave are swept in
// one straight run of code, so their gathers and sums overlap: a workgroup
// has about one wave per SIMD and nothing else hides LDS latency.  Slots past
// a slice's width hold zeros and read what res_padded says.
//
// ADJ: the reverse sweeps of the adjoint on the layout of A^T.  What is
// exchanged is mu = D^{-1} lambda; lambda takes b's place (lambda -= A^T mu),
// every mu is also stored for the gradient pass, and their sum is returned.
template <typename T, int NRHS, int W, int SPL, bool LOC, bool ADJ>
__device__ void res_tile(const ResParams& P, int32_t tile, char* smem, int32_t ldx)
{
    using U = typename Bits<T>::type;
    constexpr U SENT = Bits<T>::sentinel;
    constexpr int HU = res_halo(W);
    constexpr bool WIDE = W > 14, TABW = WIDE && !LOC;
    constexpr int NC = (W + 3) / 4;                 // groups of four positions
    constexpr int UB = NRHS == 1 ? (sizeof(T) == 8 ? (WIDE && LOC ? 1 : 2) : 4) : NRHS == 2 && sizeof(T) == 4 ? 2 : 1;   // slots per batch of gathers
    constexpr int JB = NRHS == 4 ? 1 : SPL;         // slices per batch
    constexpr bool DB = res_two_buffers(NRHS, W, LOC);
    constexpr bool BL = res_rhs_in_lds(sizeof(T), NRHS, W, LOC);
    constexpr int NW = kResBlock / 64;
    constexpr bool PAD = sizeof(T) == 8 && !ADJ;    // see res_padded
    const ResSys* const D = &P.sys;                 // kernel arguments
    const uint32_t kbase = P.kbase;
    const int32_t n = D->n;
    const int32_t r0 = ((cptr<const int32_t>)D->tile_row0)[tile], r1 = ((cptr<const int32_t>)D->tile_row0)[tile + 1];
    const int32_t s0 = ((cptr<const int32_t>)D->tile_slice0)[tile], s1 = ((cptr<const int32_t>)D->tile_slice0)[tile + 1];
    // positions count from the first entry a row reads (TABW: `under` entries before the footprint)
    const int32_t under = TABW ? D->under : 0;
    const int32_t fp = ((cptr<const int32_t>)D->fp)[tile] + under, own = ((cptr<const int32_t>)D->own)[tile] + under;
    const int32_t rows = r1 - r0;
    const int32_t nh = fp - rows + (TABW ? D->over : 0);   // entries to gather
    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // LDS: x [buffers][NRHS][ldx], control words, gather offsets, positions, b
    T* const lds_zero = reinterpret_cast<T*>(smem);
    T* const lds_x = lds_zero + (TABW ? 2 * kResPad - under : 1);
    int32_t* const lds_ctl = reinterpret_cast<int32_t*>(smem + (DB ? 2 : 1) * res_x_bytes(ldx, NRHS, sizeof(T)));
    uint32_t* const lds_hg = reinterpret_cast<uint32_t*>(lds_ctl + kResCtlWords);
    uint2* const lds_pos = reinterpret_cast<uint2*>(lds_hg + (WIDE ? HU * kResBlock : 0));   // [group][row]
    T* const lds_b = reinterpret_cast<T*>(lds_pos);                                          // (no positions then)
    const int32_t xbuf = DB ? (int32_t)(res_x_bytes(ldx, NRHS, sizeof(T)) / sizeof(T)) : 0;  // entries to the other buffer

    // footprint entries gathered from other tiles: byte offset of each in a
    // ring slot's column (the tile's runs are searched in LDS, once)
    uint32_t hg[HU];
    {
        const int32_t run0 = ((cptr<const int32_t>)D->run0)[tile];
        const int32_t nr = ((cptr<const int32_t>)D->run0)[tile + 1] - run0;
        const gptr<const int32_t> rl = (gptr<const int32_t>)D->run_lds;
        const gptr<const int32_t> rd = (gptr<const int32_t>)D->run_delta;
        int32_t* lrl = reinterpret_cast<int32_t*>(smem);
        int32_t* lrd = lrl + nr;
        for (int32_t q = tid; q < nr; q += kResBlock) {
            lrl[q] = rl[run0 + q];
            lrd[q] = rd[run0 + q];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < HU; ++u) {
            const int32_t e = min(u * kResBlock + tid, max(nh - 1, 0));
            const int32_t pos = min(max(e < own ? e : e + rows, under), fp - 1) - under;
            int32_t lo = 0, hi = nr - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (lrl[mid] <= pos) lo = mid; else hi = mid - 1;
            }
            hg[u] = (uint32_t)(pos + lrd[lo]) * (uint32_t)sizeof(T);
        }
        __syncthreads();
        if constexpr (WIDE) {
#pragma unroll
            for (int u = 0; u < HU; ++u) lds_hg[u * kResBlock + tid] = hg[u];
        }
    }

    // the tile's slots, right-hand sides, reciprocal diagonals and rows of x
    T a[SPL][W];
    uint2 cp[WIDE ? 1 : SPL][WIDE ? 1 : NC];        // positions of four slots each
    int32_t shv[TABW ? SPL : 1];                    // lane k: byte shift of slot k
    T bv[BL ? 1 : SPL][NRHS], di[SPL], xs[SPL][NRHS];
    T sum[ADJ ? SPL : 1];                           // ADJ: the sum of mu
    {
        const cptr<const int64_t> slice_off = (cptr<const int64_t>)D->slice_off;
        const cptr<const int32_t> shift = (cptr<const int32_t>)D->shift;
        const gptr<const T> val = (gptr<const T>)D->val;
        const gptr<const T> b = (gptr<const T>)D->b;
        const gptr<const T> x0 = (gptr<const T>)D->x0;
        const gptr<const uint16_t> col16 = (gptr<const uint16_t>)D->col16;
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int32_t s = s0 + wave + j * NW;
            const bool live = s < s1;
            const int64_t soff = live ? slice_off[s] : 0;
            const int32_t w = live ? (int32_t)((slice_off[s + 1] - soff) >> 6) : 0;
            const int32_t i = r0 + (s - s0) * 64 + lane;
            const int32_t ib = min(i, r1 - 1);
            T d = (T)1;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                a[j][k] = (T)0;
                if (k < w) a[j][k] = val[soff + (int64_t)k * 64 + lane];
            }
            if constexpr (TABW) {
                shv[j] = (res_wide_shift(lane, w, PAD, w > 0 ? shift[(soff >> 6) + min(lane, w - 1)] : 0,
                                         r0 + (s - s0) * 64) + under) * (int32_t)sizeof(T);
#pragma unroll
                for (int k = 0; k < W; ++k)
                    if (k < w && shift[(soff >> 6) + k] == own - under - r0 && a[j][k] != (T)0) d = a[j][k];
            } else {
#pragma unroll
                for (int q = 0; q < NC; ++q) {
                    uint32_t p4[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        constexpr int kLast = W - 1;
                        const int k = min(4 * q + u, kLast);
                        int32_t pos = -1;                           // a zero
                        if (k < res_padded(w, PAD)) {
                            const int32_t kk = min(k, w - 1);
                            if constexpr (LOC) pos = col16[soff + (int64_t)kk * 64 + lane];
                            else pos = min(max(i + shift[(soff >> 6) + kk], 0), fp - 1);
                            // the row's diagonal: the slot of its own position
                            if (k < w && pos == own + (i - r0) && a[j][k] != (T)0) d = a[j][k];
                        }
                        p4[u] = (uint32_t)(pos + 1) * (uint32_t)sizeof(T);
                    }
                    const uint2 p2 = make_uint2(p4[0] | p4[1] << 16, p4[2] | p4[3] << 16);
                    if constexpr (WIDE) lds_pos[q * (SPL * kResBlock) + j * kResBlock + tid] = p2;
                    else cp[j][q] = p2;
                }
            }
            if constexpr (ADJ) di[j] = ((gptr<const T>)D->invd)[ib];
            else di[j] = (T)1 / d;
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                if constexpr (BL) lds_b[j * kResBlock + tid] = b[(int64_t)ib * NRHS + c];
                else bv[j][c] = b[(int64_t)ib * NRHS + c];
                xs[j][c] = (T)0;
                if constexpr (ADJ) {
                    xs[j][c] = di[j] * b[ib];
                    sum[j] = xs[j][c];
                    if (i < r1) ((gptr<T>)P.xall)[(int64_t)P.kend * n + i] = xs[j][c];
                } else if (D->x0) {
                    xs[j][c] = x0[(int64_t)ib * NRHS + c];
                }
            }
        }
    }

    U* const ring = reinterpret_cast<U*>(D->ring);
    const int64_t slot = (int64_t)n * NRHS;
    ResCtl* const ctl = D->ctl;
    const bool is_max = P.norm_inf != 0;
    const int32_t nd = P.nd;
    constexpr int CT = kResBlock - 64;              // the thread that reads the control words (the last wave's first)
    uint32_t saved = 0;
    int32_t word = -1, st[NRHS];                    // last sweep seen decided, stop sweeps (negative: running)
#pragma unroll
    for (int c = 0; c < NRHS; ++c) st[c] = -1;
    // control words in LDS, by sweep parity: stop words, bit c: column c has
    // stopped; then 1: gave up
    if (tid == 0) lds_ctl[kResGaveUp] = 0;
    // the zeros that slots past a slice's width read
    if (tid < (TABW ? kResPad : 1)) {
#pragma unroll
        for (int h = 0; h < (DB ? 2 : 1); ++h)
#pragma unroll
            for (int c = 0; c < NRHS; ++c) lds_zero[h * xbuf + c * ldx + tid] = (T)0;
    }
    __syncthreads();

    // Every thread's part of x_k from the other tiles: the loads ...
    auto from = [&](int u, int32_t tv) -> uint32_t { return WIDE ? lds_hg[u * kResBlock + tv] : hg[u]; };
    auto ask = [&](const U* src, U (&v)[HU][NRHS], int32_t tv) {
#pragma unroll
        for (int u = 0; u < HU; ++u) {
            const uint32_t o = from(u, tv);
#pragma unroll
            for (int c = 0; c < NRHS; ++c) v[u][c] = ldo(src + (int64_t)c * n, o);
        }
    };
    // ... repeated until every value is there, then into LDS, beside the own rows
    auto take = [&](const U* src, U (&v)[HU][NRHS], const T (&xo)[SPL][NRHS], T* xl, int32_t tv) {
        Patience wait;
        for (;;) {
            bool miss = false;
#pragma unroll
            for (int u = 0; u < HU; ++u)
#pragma unroll
                for (int c = 0; c < NRHS; ++c) miss |= v[u][c] == SENT;
            if (!miss) break;
#pragma unroll
            for (int u = 0; u < HU; ++u)
#pragma unroll
                for (int c = 0; c < NRHS; ++c)
                    if (v[u][c] == SENT) v[u][c] = ldo(src + (int64_t)c * n, from(u, tv));
            if (wait.out(P)) {
                lds_ctl[kResGaveUp] = 1;
                break;
            }
            // its owner may have left with every column stopped
            if ((wait.n & 63u) == 0 && ldc(&ctl->done) == kbase) break;
        }
        if (nh > 0) {
#pragma unroll
            for (int u = 0; u < HU; ++u) {
                const int32_t e = min(u * kResBlock + tv, nh - 1);
                const int32_t pos = e < own ? e : e + rows;
#pragma unroll
                for (int c = 0; c < NRHS; ++c) {
                    T t;
                    __builtin_memcpy(&t, &v[u][c], sizeof(T));
                    xl[c * ldx + pos] = t;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int32_t li = tv + j * kResBlock;
            if (li < rows) {
#pragma unroll
                for (int c = 0; c < NRHS; ++c) xl[c * ldx + own + li] = xo[j][c];
            }
        }
    };
    // Columns newly stopped (stop words in LDS): this tile's rows of the
    // iterate they stopped on; true when all have.
    auto save = [&](const int32_t* lc, int32_t tv) -> bool {
#pragma unroll
        for (int c = 0; c < NRHS; ++c) {
            const int32_t sk = __builtin_amdgcn_readfirstlane(lc[c]);
            if (sk < 0 || ((saved >> c) & 1u)) continue;
            saved |= 1u << c;
            const U* from_k = ring + (int64_t)(sk % kResRing) * slot + (int64_t)c * n;
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                const int32_t li = tv + j * kResBlock;
                if (li < rows) {
                    const U t = ldo(from_k, (uint32_t)(r0 + li) * (uint32_t)sizeof(T));
                    reinterpret_cast<U*>(D->xout)[(int64_t)(r0 + li) * NRHS + c] = t;
                }
            }
        }
        return saved == (1u << NRHS) - 1u;
    };

    // this tile's share of the ring and of the partials: x_0, sentinels
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
        const int32_t li = tid + j * kResBlock;
        if (li < rows) {
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                const uint32_t o = (uint32_t)(r0 + li) * (uint32_t)sizeof(T);
                U w0;
                __builtin_memcpy(&w0, &xs[j][c], sizeof(T));
                if (w0 == SENT) w0 ^= 1;
                sto(ring + (int64_t)c * n, o, w0);
#pragma unroll
                for (int q = 1; q < kResRing; ++q) sto(ring + q * slot + (int64_t)c * n, o, (U)SENT);
            }
        }
    }
    {
        constexpr int NP = res_partials(NRHS, W, LOC) * NRHS;
        for (int32_t q = tid; q < kResPart * NP; q += kResBlock)
            stc(reinterpret_cast<uint64_t*>(D->part) + ((int64_t)(q / NP) * D->ntiles + tile) * NP + q % NP,
                (uint64_t)Bits<double>::sentinel);
    }
    if (!res_arrive(P, lds_ctl + kResGaveUp + 1)) return;
    {
        U v[HU][NRHS];
        ask(ring, v, tid);
        take(ring, v, xs, lds_x, tid);
    }
    for (int32_t k = 0;; ++k) {
        // addresses are formed anew each sweep: kept across sweeps they would
        // take some thirty registers
        int32_t tv = tid;
        asm volatile("" : "+v"(tv));
        int32_t* const lc = lds_ctl + (k & 1) * 8;
        const T* const xl = lds_x + (k & 1) * xbuf;
        const T* const xg = TABW ? xl : xl - 1;     // what gathered positions count from
        if (tid == CT && P.solve) {
            int32_t any = 0;
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                lc[c] = st[c];
                any |= (int32_t)(st[c] >= 0) << c;
            }
            lc[4] = any;
        }
        lds_barrier();
        // fin: the last residual of the loop; in solve mode its x_{k+1} is not needed
        const bool fin = P.solve ? k >= P.kend : k + 1 >= P.kend;
        const bool last = fin && !P.solve;
        const int32_t now0 = lds_ctl[kResGaveUp], now1 = P.solve ? lc[4] : 0;
        T q[SPL][NRHS];
#pragma unroll
        for (int j = 0; j < SPL; ++j)
#pragma unroll
            for (int c = 0; c < NRHS; ++c) q[j][c] = (T)0;
        // batches of gathers, each issued before the sums of the one before
        // it (the barriers keep the compiler from issuing more, for which
        // there are no registers)
#pragma unroll
        for (int j0 = 0; j0 < SPL; j0 += JB) {
            T xv[2][UB][NRHS][JB];
            uint2 p2[2][JB];
            auto positions = [&](int g, uint2 (&p)[JB]) {
                if constexpr (!TABW) {
#pragma unroll
                    for (int j = 0; j < JB; ++j) {
                        if constexpr (WIDE) {
                            p[j] = lds_pos[g * (SPL * kResBlock) + (j0 + j) * kResBlock + tv];
                        } else {
                            asm volatile("" : "+v"(cp[j0 + j][g].x), "+v"(cp[j0 + j][g].y));   // unpack anew each sweep
                            p[j] = cp[j0 + j][g];
                        }
                    }
                }
            };
            auto gather = [&](int k0, T (&x)[UB][NRHS][JB], const uint2 (&p)[JB]) {
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    if (k0 + u < W) {
#pragma unroll
                        for (int j = 0; j < JB; ++j) {
                            int32_t off;
                            if constexpr (TABW) {
                                off = (r0 + tv + (j0 + j) * kResBlock) * (int32_t)sizeof(T) +
                                      __builtin_amdgcn_readlane(shv[j0 + j], k0 + u);
                            } else {
                                const uint32_t pp = ((k0 + u) & 2) ? p[j].y : p[j].x;
                                off = (int32_t)(((k0 + u) & 1) ? pp >> 16 : pp & 0xffffu);
                            }
#pragma unroll
                            for (int c = 0; c < NRHS; ++c)
                                x[u][c][j] =
                                    *reinterpret_cast<const T*>(reinterpret_cast<const char*>(xg + c * ldx) + off);
                        }
                    }
            };
            positions(0, p2[0]);
            if (NC > 1) positions(1, p2[1]);
            gather(0, xv[0], p2[0]);
#pragma unroll
            for (int b = 0; b * UB < W; ++b) {
                const int k1 = (b + 1) * UB;
                if (k1 < W) {
                    gather(k1, xv[(b + 1) & 1], p2[(k1 / 4) & 1]);
                    // the group after the one just entered
                    if (k1 % 4 == 0 && k1 / 4 + 1 < NC) positions(k1 / 4 + 1, p2[(k1 / 4 + 1) & 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    if (b * UB + u < W) {
#pragma unroll
                        for (int c = 0; c < NRHS; ++c)
#pragma unroll
                            for (int j = 0; j < JB; ++j) {
                                const T x = xv[b & 1][u][c][j], m = a[j0 + j][b * UB + u];
                                if constexpr (sizeof(T) == 8) q[j0 + j][c] = __builtin_fma(m, x, q[j0 + j][c]);
                                else q[j0 + j][c] = __builtin_fmaf(m, x, q[j0 + j][c]);
                                // the per-sweep launches' batch ends one slot further
                                if constexpr (PAD && W % 7 != 0)
                                    if (b * UB + u == W - 1) q[j0 + j][c] = __builtin_fma((T)0, x, q[j0 + j][c]);
                            }
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
            // the sums stay here (the compiler would move them past the exits below, gathered values and all)
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int c = 0; c < NRHS; ++c) asm volatile("" : "+v"(q[j0 + j][c]));
        }
        {
            const int32_t gave_up = __builtin_amdgcn_readfirstlane(now0), stopped = __builtin_amdgcn_readfirstlane(now1);
            if (gave_up != 0) return;
            if ((uint32_t)stopped != saved && save(lc, tv)) return;
        }
        double rd[SPL][NRHS];                       // residuals, 0 past the tile's last row
        U* dst = ring + (int64_t)((k + 1) % kResRing) * slot;
        // the rows' own x_k comes from LDS: held in registers it would be
        // live beside the gathers
        T xo[SPL][NRHS];
#pragma unroll
        for (int j = 0; j < SPL; ++j)
#pragma unroll
            for (int c = 0; c < NRHS; ++c) xo[j][c] = xl[c * ldx + min(own + tv + j * kResBlock, fp - 1)];
        wait_own();                                 // the sentinels of sweep k + 2 are in place
        asm volatile("" : "+v"(word));              // loaded a sweep ago: taken here, not behind this sweep's stores
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int32_t li = tv + j * kResBlock;
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                const T r = (BL ? lds_b[j * kResBlock + tv] : bv[BL ? 0 : j][c]) - q[j][c];
                if constexpr (ADJ) {
                    if constexpr (BL) lds_b[j * kResBlock + tv] = r;
                    else bv[j][c] = r;
                    xo[j][c] = di[j] * r;
                    sum[j] = __builtin_fma(di[j], r, sum[j]);   // as the per-step kernel contracts it
                    rd[j][c] = 0.0;
                } else {
                    xo[j][c] = xo[j][c] + di[j] * r;
                    rd[j][c] = li < rows ? (double)r : 0.0;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int32_t li = tv + j * kResBlock;
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                U w2;
                __builtin_memcpy(&w2, &xo[j][c], sizeof(T));
                if (w2 == SENT) w2 ^= 1;            // never publish the sentinel itself
                if (li < rows) sto(dst + (int64_t)c * n, (uint32_t)(r0 + li) * (uint32_t)sizeof(T), w2);
            }
        }
        // iterates kept by the caller: x_{k+1}, or mu counted downwards
        if (NRHS == 1 && sizeof(T) == 8 && P.xall) {
            T* const keep = static_cast<T*>(P.xall) + (int64_t)(ADJ ? P.kend - 1 - k : k + 1) * n;
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                const int32_t li = tv + j * kResBlock;
                if (li < rows) __builtin_nontemporal_store(xo[j][0], (gptr<T>)keep + (r0 + li));
            }
        }
        // the wave's norm partial
        double acc[NRHS];
#pragma unroll
        for (int c = 0; c < NRHS; ++c) acc[c] = 0.0;
        if (is_max) {
#pragma unroll
            for (int j = 0; j < SPL; ++j)
#pragma unroll
                for (int c = 0; c < NRHS; ++c) acc[c] = maxnan(acc[c], fabs(rd[j][c]));
            wave_reduce<true>(acc);
        } else {
#pragma unroll
            for (int j = 0; j < SPL; ++j)
#pragma unroll
                for (int c = 0; c < NRHS; ++c) acc[c] = __builtin_fma(rd[j][c], rd[j][c], acc[c]);
            wave_reduce<false>(acc);
        }
        U v[HU][NRHS];
        if (!fin) {
            // For sweep k + 1: sweep k + 4 - ring has to be decided (its slot
            // is cleared then), the stop words are read after that was seen;
            // every thread asks for its part of x_{k+1}.  Asked for with a
            // delay: another tile's store needs some 0.4 us to be seen, and a
            // try that comes before it costs its whole trip and leaves the
            // line in this XCD's L2, which the store then has to take back
            // (fixed sweeps without the pause and with it: 20^3 1.86 and 1.91
            // us, 33^3 2.08 and 1.94, 64^3 3.23 and 3.14, 80^3 5.13 and 4.85).
            if (tid == CT) {
                const int32_t need = k + 4 - kResRing;
                if (need >= 0 && word < need) {
                    Patience wait;
                    for (;;) {
                        word = (int32_t)(ldc(&ctl->word[need & (nd - 1)]) - kbase);
                        if (word >= need || ldc(&ctl->done) == kbase) break;
                        if (wait.out(P)) {
                            lds_ctl[kResGaveUp] = 1;
                            break;
                        }
                    }
                }
                asm volatile("" ::: "memory");
                if (P.solve) {
#pragma unroll
                    for (int c = 0; c < NRHS; ++c) st[c] = (int32_t)(ldc(&ctl->stop[c]) - kbase);
                }
                word = (int32_t)(ldc(&ctl->word[max(need + 1, 0) & (nd - 1)]) - kbase);
            }
            __builtin_amdgcn_s_sleep(10);           // 10 * 64 cycles
            ask(dst, v, tv);
            U* clr = ring + (int64_t)((k + 3) % kResRing) * slot;
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                const int32_t li = tv + j * kResBlock;
                if (li < rows) {
#pragma unroll
                    for (int c = 0; c < NRHS; ++c)
                        sto(clr + (int64_t)c * n, (uint32_t)(r0 + li) * (uint32_t)sizeof(T), (U)SENT);
                }
            }
        }
        uint64_t* part = reinterpret_cast<uint64_t*>(D->part) +
                         ((int64_t)(k % kResPart) * D->ntiles + tile) * (res_partials(NRHS, W, LOC) * NRHS);
        if constexpr (DB) {
            // no barrier here: the deciding workgroups add the waves' partials
            if (lane == 0) {
                uint64_t w = (uint64_t)__double_as_longlong(acc[0]);
                if (w == Bits<double>::sentinel) w ^= 1;
                stc(&part[wave], w);
            }
        } else {
            double* red = reinterpret_cast<double*>(lds_ctl + kResCtlWords - 2 * kResRed);
            if (lane == 0) {
#pragma unroll
                for (int c = 0; c < NRHS; ++c) red[c * NW + wave] = acc[c];
            }
            lds_barrier();                          // also: every read of lds_x is done
            if (tv < NRHS) {
                double s = red[tv * NW];
#pragma unroll
                for (int w = 1; w < NW; ++w) s = is_max ? maxnan(s, red[tv * NW + w]) : s + red[tv * NW + w];
                uint64_t w = (uint64_t)__double_as_longlong(s);
                if (w == Bits<double>::sentinel) w ^= 1;
                stc(&part[tv], w);
            }
        }
        if (last) {
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                const int32_t li = tv + j * kResBlock;
                if (li < rows) {
#pragma unroll
                    for (int c = 0; c < NRHS; ++c)
                        reinterpret_cast<T*>(D->xout)[(int64_t)(r0 + li) * NRHS + c] = ADJ ? sum[ADJ ? j : 0] : xo[j][c];
                }
            }
            return;
        }
        if (fin) break;
        take(dst, v, xo, lds_x + ((k + 1) & 1) * xbuf, tv);
    }
    // at the last residual every column stops
    __syncthreads();
    if (tid == 0) {
        Patience wait;
        while (ldc(&ctl->done) != kbase)
            if (wait.out(P)) {
                lds_ctl[kResGaveUp] = 1;
                break;
            }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int c = 0; c < NRHS; ++c) lds_ctl[c] = (int32_t)(ldc(&ctl->stop[c]) - kbase);
    }
    __syncthreads();
    if (lds_ctl[kResGaveUp] == 0) save(lds_ctl, tid);
}

// Waves per SIMD asked of the compiler: what the registers held across a
// sweep leave room for, some at the price of a spill (14 registers in the
// FP64 four-column 7-slot kernels, 4 in the 27-slot adjoint, 2 and 1 in the
// FP32 27-slot ones, 1 in the FP64 27-slot table kernel).
template <typename T>
constexpr int res_waves(int nrhs, int w, bool loc, bool adj)
{
    if (sizeof(T) == 8) return nrhs == 1 ? (w <= 7 ? (adj ? 4 : 5) : 3) : nrhs == 2 ? (w <= 7 ? 4 : 2) : w <= 7 ? 3 : 1;
    return nrhs == 1 ? (w <= 7 ? 7 : 5) : nrhs == 2 ? (w <= 7 ? 5 : 4) : w <= 7 ? 4 : 2;
}

template <typename T, int NRHS, int W, int SPL, bool LOC, bool ADJ>
__global__ void __launch_bounds__(kResBlock) __attribute__((amdgpu_waves_per_eu(res_waves<T>(NRHS, W, LOC, ADJ))))
k_resident(ResParams P, int32_t ldx)
{
    extern __shared__ __align__(16) char smem[];
    // neighbouring tiles on one XCD, then the deciding workgroups
    const int32_t wg = (int32_t)blockIdx.x, ntiles = P.sys.ntiles;
    if (wg >= ntiles) {
        if (wg == ntiles && threadIdx.x == 0) {
            stc(&P.sys.ctl->status, (int32_t)JAC_OK);
            stc(&P.sys.ctl->last_k, -1);
            __hip_atomic_store(&P.seen->started, P.kbase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            stc(&P.sys.ctl->redo_sweeps, 0u);
            stc(&P.sys.ctl->redo_next, (uint64_t)0);
            stc(&P.sys.ctl->redo_done, (uint64_t)0);
        }
        int32_t* ok = reinterpret_cast<int32_t*>(smem);
        if (!res_arrive(P, ok)) return;
        __syncthreads();
        res_decide<NRHS, res_partials(NRHS, W, LOC)>(P, wg - ntiles, reinterpret_cast<double*>(smem));
        return;
    }
    int32_t first, end, stride;
    xcd_items(ntiles, ntiles, wg, first, end, stride);
    res_tile<T, NRHS, W, SPL, LOC, ADJ>(P, first, smem, ldx);
}

// Closes a launch of fixed FP64 sweeps the host does not wait for: copies
// x_K to its place and reports to the host, or, if the launch gave up, does
// its sweeps again from x0, which is still intact: iterates, norms and kept
// iterates to the bit, with nothing asked of the workgroups' residency.
// Workgroups take (sweep, tile) items in order from a counter, and an item
// waits for the end of the sweep before: every item it can wait for was taken
// by a workgroup that is running, so each wait ends.  (x in two ring slots,
// columns searched through the footprint's runs: some 60 us a sweep at 65^3
// would do, and this one never has to be fast.)
template <int NRHS>
__global__ void __launch_bounds__(kResBlock) k_res_finish(ResParams P, int32_t loc, int32_t max_runs, double* x0_out)
{
    extern __shared__ __align__(16) char smem[];
    __shared__ double red[kResRed];
    __shared__ uint64_t item_;
    __shared__ int32_t last_;
    const ResSys& S = P.sys;
    ResCtl* ctl = S.ctl;
    const int32_t n = S.n;
    const bool gave_up = ldc(&ctl->abort) == P.kbase;
    ResSeen* seen = P.seen;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // host memory: plain loads and stores; launches of one stream, so one writer at a time
        if (gave_up)
            __hip_atomic_store(&seen->gave_up, __hip_atomic_load(&seen->gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) + 1,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&seen->ended, P.kbase, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (!gave_up) {
        const int64_t m = (int64_t)n * NRHS;
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
            x0_out[i] = static_cast<const double*>(S.xout)[i];
        return;
    }
    int32_t* lrl = reinterpret_cast<int32_t*>(smem);
    int32_t* lrd = lrl + max_runs;
    const int32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t total = (uint64_t)P.kend * (uint64_t)S.ntiles;
    const double* val = static_cast<const double*>(S.val);
    const double* b = static_cast<const double*>(S.b);
    const double* x0 = static_cast<const double*>(S.x0);
    for (;;) {
        if (tid == 0)
            item_ = __hip_atomic_fetch_add(&ctl->redo_next, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const uint64_t item = item_;
        if (item >= total) return;
        const int32_t k = (int32_t)(item / (uint64_t)S.ntiles), tile = (int32_t)(item % (uint64_t)S.ntiles);
        if (tid == 0)
            while (ldc(&ctl->redo_sweeps) < (uint32_t)k) __builtin_amdgcn_s_sleep(16);
        const int32_t run0 = S.run0[tile], nr = S.run0[tile + 1] - run0;
        for (int32_t q = tid; q < nr; q += kResBlock) {
            lrl[q] = S.run_lds[run0 + q];
            lrd[q] = S.run_delta[run0 + q];
        }
        __syncthreads();
        const double* from = static_cast<const double*>(S.ring) + (int64_t)(k & 1) * n * NRHS;
        double* to = static_cast<double*>(S.ring) + (int64_t)((k + 1) & 1) * n * NRHS;
        auto x_at = [&](int32_t i, int c) -> double {
            if (k == 0) return x0 ? x0[(int64_t)i * NRHS + c] : 0.0;
            return ldc(&from[(int64_t)c * n + i]);
        };
        const int32_t r0 = S.tile_row0[tile], r1 = S.tile_row0[tile + 1];
        const int32_t s0 = S.tile_slice0[tile], s1 = S.tile_slice0[tile + 1];
        const int32_t fp = S.fp[tile], own = S.own[tile];
        double acc[NRHS];
#pragma unroll
        for (int c = 0; c < NRHS; ++c) acc[c] = 0.0;
        for (int32_t s = s0 + wave; s < s1; s += kResBlock / 64) {
            const int64_t soff = S.slice_off[s];
            const int32_t w = (int32_t)((S.slice_off[s + 1] - soff) >> 6);
            const int32_t i = r0 + (s - s0) * 64 + lane;
            if (i >= r1) continue;
            double q[NRHS], d = 1.0;
#pragma unroll
            for (int c = 0; c < NRHS; ++c) q[c] = 0.0;
            for (int32_t e = 0; e < res_padded(w, true); ++e) {
                const int32_t ee = min(e, w - 1);
                const int64_t slot = soff + (int64_t)ee * 64 + lane;
                const double a = e < w ? val[slot] : 0.0;
                const int32_t pos = loc ? (int32_t)S.col16[slot] : min(max(i + S.shift[(soff >> 6) + ee], 0), fp - 1);
                const bool diag = loc ? pos == own + (i - r0) : S.shift[(soff >> 6) + ee] == own - r0;
                int32_t lo = 0, hi = nr - 1;
                while (lo < hi) {
                    const int32_t mid = (lo + hi + 1) >> 1;
                    if (lrl[mid] <= pos) lo = mid; else hi = mid - 1;
                }
                const int32_t col = pos + lrd[lo];
#pragma unroll
                for (int c = 0; c < NRHS; ++c) q[c] = __builtin_fma(a, x_at(col, c), q[c]);
                if (diag && a != 0.0) d = a;
            }
            const double di = 1.0 / d;
#pragma unroll
            for (int c = 0; c < NRHS; ++c) {
                const double r = b[(int64_t)i * NRHS + c] - q[c];
                const double x = __builtin_fma(di, r, x_at(i, c));
                stc(&to[(int64_t)c * n + i], x);
                if (k + 1 == P.kend) x0_out[(int64_t)i * NRHS + c] = x;
                if (NRHS == 1 && P.xall) static_cast<double*>(P.xall)[(int64_t)(k + 1) * n + i] = x;
                acc[c] = __builtin_fma(r, r, acc[c]);
            }
        }
        wait_own();
        block_reduce<NRHS>(acc, false, red);        // its barriers: every wave's stores have reached the device
        double* part = S.part + (int64_t)(k & 1) * S.ntiles * NRHS;
        if (tid == 0) {
#pragma unroll
            for (int c = 0; c < NRHS; ++c) stc(&part[(int64_t)tile * NRHS + c], acc[c]);
            wait_own();
            last_ = (__hip_atomic_fetch_add(&ctl->redo_done, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1) %
                        (uint64_t)S.ntiles == 0;
        }
        __syncthreads();
        if (last_) {
            // the sweep's last tile: its norm, in the order of the other loops, before the next sweep starts
            double v[NRHS];
#pragma unroll
            for (int c = 0; c < NRHS; ++c) v[c] = 0.0;
            for (int32_t t = tid; t < S.ntiles; t += kResBlock)
#pragma unroll
                for (int c = 0; c < NRHS; ++c) v[c] = v[c] + ldc(&part[(int64_t)t * NRHS + c]);
            block_reduce<NRHS>(v, false, red);
            if (tid == 0) {
#pragma unroll
                for (int c = 0; c < NRHS; ++c)
                    if (P.hist) P.hist[(int64_t)k * NRHS + c] = sqrt(v[c]);
                stc(&ctl->redo_sweeps, (uint32_t)k + 1);
            }
        }
        // Thread 0's branch above and its claim of the next item must not meet
        // across the loop's end: the compiler then threads one into the other
        // and sends the other threads round a loop of their own, past the
        // barrier, on the old item.
        __syncthreads();
    }
}

template <typename U>
__global__ void __launch_bounds__(256) k_res_settle(const U* __restrict__ from, U* __restrict__ to, int64_t m,
                                                    const ResCtl* __restrict__ ctl, uint32_t kbase, bool more)
{
    if (ctl->abort == kbase || (more && ctl->status == JAC_NOT_CONVERGED)) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        to[i] = from[i];
}

template <typename T, int NRHS, int W, int SPL>
void* pick_loc(bool loc)
{
    return loc ? reinterpret_cast<void*>(&k_resident<T, NRHS, W, SPL, true, false>)
               : reinterpret_cast<void*>(&k_resident<T, NRHS, W, SPL, false, false>);
}
template <typename T, int NRHS>
void* pick_shape(int width, int slices, bool loc)
{
    if (slices <= 2) {
        if (width <= 7) return pick_loc<T, NRHS, 7, 2>(loc);
        if (width <= 14) return pick_loc<T, NRHS, 14, 2>(loc);
        if (width <= 27) return pick_loc<T, NRHS, 27, 2>(loc);
    }
    return nullptr;
}
template <typename T>
void* pick_rhs(int nrhs, int width, int slices, bool loc)
{
    switch (nrhs) {
    case 1: return pick_shape<T, 1>(width, slices, loc);
    case 2: return pick_shape<T, 2>(width, slices, loc);
    case 4: return pick_shape<T, 4>(width, slices, loc);
    default: return nullptr;
    }
}

}  // namespace

void* res_adjoint_kernel(int width, int slices)
{
    if (slices > 2) return nullptr;
    if (width <= 7) return reinterpret_cast<void*>(&k_resident<double, 1, 7, 2, false, true>);
    if (width <= 14) return reinterpret_cast<void*>(&k_resident<double, 1, 14, 2, false, true>);
    if (width <= 27) return reinterpret_cast<void*>(&k_resident<double, 1, 27, 2, false, true>);
    return nullptr;
}

void* res_kernel(bool fp32, int nrhs, int width, int slices, bool explicit_cols)
{
    return fp32 ? pick_rhs<float>(nrhs, width, slices, explicit_cols)
                : pick_rhs<double>(nrhs, width, slices, explicit_cols);
}

hipError_t launch_res(void* fn, int grid, size_t lds, int32_t ldx, hipStream_t st, ResParams p, bool cooperative)
{
    void* args[] = {&p, &ldx};
    if (cooperative) return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kResBlock), args, (unsigned)lds, st);
    return hipLaunchKernel(fn, dim3(grid), dim3(kResBlock), args, lds, st);
}

void launch_res_finish(int nrhs, bool loc, int32_t runs, hipStream_t st, ResParams p, double* x0)
{
    const int64_t m = (int64_t)p.sys.n * nrhs;
    const int g = (int)std::min<int64_t>((m + kResBlock - 1) / kResBlock, 2048);
    const size_t lds = (size_t)runs * 8;
    if (nrhs == 1) k_res_finish<1><<<g, kResBlock, lds, st>>>(p, loc, runs, x0);
    else if (nrhs == 2) k_res_finish<2><<<g, kResBlock, lds, st>>>(p, loc, runs, x0);
    else k_res_finish<4><<<g, kResBlock, lds, st>>>(p, loc, runs, x0);
    JAC_HIP(hipGetLastError());
}

void launch_res_settle(bool fp32, hipStream_t st, const void* xout, void* x0, int64_t m, const ResCtl* ctl,
                       uint32_t kbase, bool more)
{
    const int g = (int)std::min<int64_t>(std::max<int64_t>((m + 255) / 256, 1), 2048);
    if (fp32)
        k_res_settle<<<g, 256, 0, st>>>(static_cast<const uint32_t*>(xout), static_cast<uint32_t*>(x0), m, ctl, kbase,
                                            more);
    else
        k_res_settle<<<g, 256, 0, st>>>(static_cast<const uint64_t*>(xout), static_cast<uint64_t*>(x0), m, ctl, kbase,
                                            more);
    JAC_HIP(hipGetLastError());
}

}  // namespace jac
