// Resident sweep loop: device structures and launchers (resident.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"

namespace jac {

constexpr int kResBlock = 256;      // threads per workgroup: the norm's summation order is that of 256-thread launches
constexpr int kResRing = 8;         // iterates in flight: x_k lives in ring slot k mod 8
constexpr int kResPart = 16;        // norm partials in flight, by sweep mod 16
// Footprint entries of other tiles a thread gathers per sweep, at most: a
// 512-row tile of a 7-point row's matrix has up to 1280 of them on planes of
// 128 x 128 nodes, of a 27-point row's up to 1606 on 96 x 96.
constexpr int res_halo(int width) { return width <= 7 ? 5 : 7; }
constexpr int kResDeciders = 4;     // deciding workgroups of a single system (sweep k is decided by number k mod 4)

constexpr int kResRed = 16;         // doubles of reduction scratch (deciding workgroups); 8 control words follow
constexpr int kResGaveUp = 16;
constexpr int kResCtlWords = 20 + 2 * kResRed;   // control words and scratch of a tile in LDS

// Bytes of x in LDS: ldx entries per right-hand side.
constexpr size_t res_x_bytes(size_t ldx, size_t nrhs, size_t elem) { return (ldx * nrhs * elem + 15) / 16 * 16; }

// Two x buffers in LDS (one barrier per sweep instead of two) where that does
// not cost a workgroup per CU.
constexpr bool res_two_buffers(int nrhs, int width, bool loc) { return nrhs == 1 && !(loc && width > 14); }
// Norm partials a tile stores per sweep and right-hand side: one per wave
// where the tile has no barrier to add them behind.
constexpr int res_partials(int nrhs, int width, bool loc) { return res_two_buffers(nrhs, width, loc) ? kResBlock / 64 : 1; }
// b in LDS instead of registers: the FP64 27-point table kernel is four registers short without.
constexpr bool res_rhs_in_lds(size_t elem, int nrhs, int width, bool loc)
{
    return elem == 8 && nrhs == 1 && width > 14 && !loc;
}

// A slot past a slice's width holds a zero value, and what x it multiplies
// matters where x is infinite or NaN: as in the per-sweep launches, up to the
// next multiple of their batch it is the slice's last slot's (FP64 sweeps;
// the FP32 ones and the adjoint's steps stop at the width).  The slots beyond
// read a zero.
constexpr int res_padded(int w, bool batched) { return batched ? (w + 6) / 7 * 7 : w; }

// The wide shift-table kernels read LDS at row plus shift without a clamp: up
// to kResPad entries before the footprint hold its first entry, up to kResPad
// behind it the last one (what the per-sweep launches' clamp reads for rows
// without an entry of the shift), and kResPad zeros come before all.
constexpr int32_t kResPad = 64;
// Entries of LDS such a tile takes beside its footprint.
constexpr int32_t kResEnds = 3 * kResPad;
// Shift that puts the 64 lanes of a slice whose first row is row0 on the
// zeros: slots past the width, and all slots of a slice the tile does not
// have (a wave's second slice, past the tile's end).
constexpr int32_t res_zero_shift(int32_t row0) { return -row0 - 2 * kResPad; }
// Shift of slot k of a slice of w slots; last is the table's shift of slot min(k, w - 1).
constexpr int32_t res_wide_shift(int k, int w, bool batched, int32_t last, int32_t row0)
{
    return k < res_padded(w, batched) ? last : res_zero_shift(row0);
}

// Control words of one system, exchanged by its workgroups during a launch.
// Sweep k of a launch is written as kbase + k, with a kbase beyond every
// sweep of the launches before, so what an earlier launch left reads as "not
// yet" and no launch has to reset them.  That holds for words less than 2^31
// older than kbase: ResNumbers says when they are zeroed.
struct ResCtl {
    uint32_t word[8];               // last sweep each deciding workgroup has decided
    uint32_t stop[4];               // column stopped on the residual of this sweep
    uint32_t done;                  // kbase of the launch: every column has stopped
    uint32_t abort;                 // kbase of the launch: a wait ran out, every workgroup leaves
    uint32_t arrived;               // workgroups that have cleared their share of the ring, all launches
    int32_t status;                 // JAC_OK, JAC_NOT_CONVERGED, JAC_E_DIVERGED
    int32_t last_k;                 // last sweep that stopped a column
    uint32_t redo_sweeps;           // fixed sweeps done again after a launch that gave up (see k_res_finish):
    double nrm[4];                  // norm of the returned iterate per column
    uint64_t redo_next;             // ... the next (sweep, tile) to take, and those done
    uint64_t redo_done;
};

// What the host learns of launches without waiting for them (pinned memory).
struct ResSeen {
    uint32_t started;               // kbase of the last launch that started
    uint32_t ended;                 // kbase of the last launch that ended
    uint32_t gave_up;               // launches that gave up
};

// The numbers a handle's launches give their sweeps and arrivals.
struct ResNumbers {
    static constexpr uint32_t kLimit = 1u << 30;
    uint32_t next = kResPart;       // number of the next launch's first sweep; zeroed words are older
    uint32_t arrived = 0;           // workgroups that all launches so far have started
    // Before a launch: true when the control words have to be zeroed first
    // (stop[] is written by solves alone, and fixed sweeps advance the
    // numbers too).
    bool restart()
    {
        if (next <= kLimit) return false;
        *this = ResNumbers();
        return true;
    }
    // The words were zeroed for another reason (a new buffer): numbers go on,
    // so that a launch is never taken for an earlier one that had its number.
    void zeroed() { arrived = 0; }
    // After a launch whose last sweep was number `last`: the tiles ran ahead
    // of it by less than kResPart sweeps.
    void passed(int32_t last) { next += (uint32_t)last + 2 * kResPart; }
};

// When a handle whose launch gave up or was refused tries again: after 32
// loops as per-sweep launches, twice as many after each further failure, up
// to 1024; at once after a success.
struct ResRetry {
    int32_t skip = 0, next = 32;
    bool now()
    {
        if (skip == 0) return true;
        --skip;
        return false;
    }
    void failed()
    {
        skip = next;
        next = next < 1024 ? 2 * next : 1024;
    }
    void ran() { next = 32; }
};

// One system of a resident launch (kernel argument).
struct ResSys {
    const int32_t* tile_row0;
    const int32_t* tile_slice0;
    const int64_t* slice_off;
    const int32_t* run0;            // footprint runs per tile: first LDS position, global column minus LDS position
    const int32_t* run_lds;
    const int32_t* run_delta;
    const int32_t* fp;              // footprint entries per tile
    const int32_t* own;             // LDS position of the tile's first row
    const int32_t* shift;           // shift-table splits: LDS position minus row, per slot column
    const uint16_t* col16;          // explicit splits: LDS position per slot
    const void* val;                // slot values, T
    const void* b;                  // T, node-major [n][nrhs] (adjoint: lambda_K)
    const void* invd;               // adjoint: D^{-1}
    const void* x0;                 // starting iterate, T (null: zero)
    void* xout;                     // returned iterate, T
    void* ring;                     // T [kResRing][nrhs][n]: iterates as their tiles publish them
    double* part;                   // [kResPart][ntiles][res_partials][nrhs]
    ResCtl* ctl;
    int32_t n, ntiles;
    int32_t under, over;            // wide shift tables: entries read before and behind the footprint
    double thr[4];
    double big[4];
};

struct ResParams {
    ResSys sys;
    double* hist;                   // nullable, [k * nrhs + c]
    // nullable: every iterate, x_k at k * n (fixed sweeps of one FP64 column);
    // adjoint: mu of the kend + 1 steps, the first (mu_K) last
    void* xall;
    ResSeen* seen;
    uint32_t kbase;                 // see ResCtl
    uint32_t arrive;                // ctl->arrived once every workgroup of this launch has arrived
    uint32_t wait;                  // longest wait for another workgroup, in ticks of the 100 MHz clock
    int32_t nd;                     // deciding workgroups (1, 2, 4 or 8)
    int32_t kend, solve, norm_inf;
};

// Kernel for up to 7, 14 or 27 slots per row and up to two slices per wave, or null when there is none.
void* res_kernel(bool fp32, int nrhs, int width, int slices, bool explicit_cols);
// Reverse sweeps of the adjoint (FP64, one column, shift table).
void* res_adjoint_kernel(int width, int slices);
// ldx: x entries in LDS per right-hand side; lds: see res_lds in resident.cpp
hipError_t launch_res(void* fn, int grid, size_t lds, int32_t ldx, hipStream_t st, ResParams p, bool cooperative);
// After a launch of fixed FP64 sweeps: x0 = xout, or, if it gave up, its
// sweeps again (loc: explicit LDS positions; runs: largest number of
// footprint runs of a tile).
void launch_res_finish(int nrhs, bool loc, int32_t runs, hipStream_t st, ResParams p, double* x0);
// After a solve: x0 = xout unless the launch gave up or, with more sweeps to
// follow in another launch, ran out of its own.
void launch_res_settle(bool fp32, hipStream_t st, const void* xout, void* x0, int64_t m, const ResCtl* ctl,
                       uint32_t kbase, bool more);

}  // namespace jac
