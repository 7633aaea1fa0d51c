// fvna_step.hpp -- the step kernels of libfvna: one launch = one attempted
// time step over every tile of one simulation (k_step) or of many
// simulations (k_step_batch).  The per-tile work is march_tile of
// fvna_device.hpp.
#pragma once

#include "fvna_device.hpp"

namespace fvna {

// Waves per SIMD the register allocation must allow: three for FP32 compute
// (134 to 139 VGPRs; with tiles that fill every slot in one round this
// measured 9% faster than four waves at 128 VGPRs on a 4096^2 grid and level
// on 8192^2), two for FP64.
#ifndef FVNA_F32_WAVES_PER_SIMD
#define FVNA_F32_WAVES_PER_SIMD 3
#endif
template <typename T> struct Occupancy { static constexpr int waves = sizeof(T) == 8 ? 2 : FVNA_F32_WAVES_PER_SIMD; };

// Workgroups are handed to the XCDs round-robin (block b to XCD b mod 8,
// each with its own L2).  Block b is given logical block start(x) + b / 8 of
// XCD x = b mod 8, so every XCD works on one contiguous run of tiles, which
// in row-major tile order is a band of whole segment rows: the halo columns
// of side-by-side strips and the warm-up rows of stacked segments are then
// read into the same L2.  A bijection of block indices; results do not
// depend on it.
constexpr int XCDS = 8;
__device__ __forceinline__ int xcd_block(int b, int nblocks)
{
    const int x = b % XCDS, k = b / XCDS;
    const int per = nblocks / XCDS, rem = nblocks % XCDS;
    return x * per + min(x, rem) + k;
}

// One attempted step over the whole grid.  force = 1 (timing): run even when
// no step is owed.
// pos = 0: the attempt runs with the clock as it stands and its CFL maximum
// goes to the clock.  pos >= 1 (the attempts of a run after its first): the
// attempt first takes the decision on the attempt before it itself.  Every wavefront computes it (control_next)
// from that attempt's clock state -- the clock for pos = 1, shadow copy
// (pos - 1) mod 2 after -- and its CFL slot (pos - 1) mod 3, none of which
// this launch writes; the grid's first wavefront stores the result as shadow
// copy pos mod 2 when its tile is done (step_end); this attempt's maximum
// goes to slot pos mod 3.  Every attempt (pos 0 included) clears slot
// (pos + 1) mod 3 for the one after it.  A closing k_ctrl_fold takes the last
// decision of the run into the clock.
//
// The words are read through the constant address space (scalar loads: no
// launch reads what it writes), and a wavefront forms only the parts of the
// decision it needs; the CFL statistics, two divisions more, are formed once,
// by the wavefront that stores them, after its tile.  With every wavefront
// forming all of it from vector loads the prologue of a 16-wavefront block
// took 4000 to 10000 cycles.
typedef const __attribute__((address_space(4))) Clock* ConstClock;
typedef const __attribute__((address_space(4))) unsigned long long* ConstU64;
typedef const __attribute__((address_space(4))) unsigned int* ConstU32;

__device__ __forceinline__ Clock read_clock(const Clock* p)
{
    const ConstClock c = (ConstClock)p;
    Clock h;
    h.t = c->t; h.dt = c->dt; h.accepted = c->accepted; h.target = c->target; h.rejected = c->rejected;
    h.attempts = c->attempts; h.status_step = c->status_step; h.smax_bits = 0; h.flags = 0; h.cur = c->cur;
    h.status = c->status; h.retries = c->retries; h.nu_last = c->nu_last; h.nu_mean = c->nu_mean;
    h.nu_m2 = c->nu_m2; h.nu_count = c->nu_count; h.x_off = c->x_off; h.pad = 0.0;
    return h;
}

// Clock state the attempt at `pos` runs with; owed: steps requested by this run
// of attempts and not yet in the clock's target (a launch that adds them to
// the clock is saved).
// (D: the simulation's descriptor, two- or three-dimensional.)
template <typename D>
__device__ __forceinline__ Clock step_clock(const D& d, int pos, long long owed)
{
    Clock* clk = d.clk;
    Clock h = read_clock(pos <= 1 ? clk : &clock_aux(clk)->shadow[(pos - 1) & 1]);
    if (pos <= 1) h.target += owed;
    if (pos == 0) return h;
    unsigned long long* psb;
    unsigned int* pfl;
    cfl_slot(clk, (pos - 1) % 3, psb, pfl);
    const unsigned long long sb = *(ConstU64)psb;
    const unsigned fl = *(ConstU32)pfl;
    // every word the decision branches on is here before its first branch: one
    // round trip to memory instead of one per branch
    asm volatile("" ::"s"(sb), "s"(fl), "s"(h.accepted), "s"(h.target), "s"(h.status), "s"(h.retries), "s"(h.cur),
                 "s"(h.dt), "s"(h.t), "s"(h.x_off));
    return control_next(h, sb, fl, d.fixed_dt, d.cfl_target, d.cfl_max, d.max_retries, 2);
}

template <typename D>
__device__ __forceinline__ bool step_begin(const D& d, int force, int pos, long long owed, Attempt& at)
{
    const Clock h = step_clock(d, pos, owed);
    unsigned long long* sb;
    unsigned int* fl;
    cfl_slot(d.clk, pos % 3, sb, fl);
    at = attempt_of(h, sb, fl);
    return force || (h.status == 0 && h.accepted < h.target);
}

// For the further kernels of an attempt: the state its first kernel (which ran
// step_begin and, in its step_end, stored the decision) ran with.
template <typename D>
__device__ __forceinline__ bool step_again(const D& d, int force, int pos, long long owed, Attempt& at)
{
    Clock h = read_clock(pos == 0 ? d.clk : &clock_aux(d.clk)->shadow[pos & 1]);
    if (pos == 0) h.target += owed;
    unsigned long long* sb;
    unsigned int* fl;
    cfl_slot(d.clk, pos % 3, sb, fl);
    at = attempt_of(h, sb, fl);
    return force || (h.status == 0 && h.accepted < h.target);
}

// By one lane of the grid: this attempt's clock state for the attempt after
// it, and a cleared CFL slot for that one to accumulate into (slot 1 after an
// attempt at pos 0).
template <typename D>
__device__ __forceinline__ void step_end(const D& d, int pos, long long owed)
{
    if (pos >= 1) clock_aux(d.clk)->shadow[pos & 1] = step_clock(d, pos, owed);
    unsigned long long* nsb;
    unsigned int* nfl;
    cfl_slot(d.clk, (pos + 1) % 3, nsb, nfl);
    *nsb = 0ull;
    *nfl = 0u;
}

// Closing decision of a run of attempts 0 .. last, each of which but the first
// took the decision on the one before it in its prologue (k_step, pos >= 1):
// the decision on attempt `last` from its clock state (the clock itself for
// last = 0) and its CFL slot goes into the clock, and every CFL slot is
// cleared for the next run.  owed: as the attempts got it.
template <typename D>
__device__ __forceinline__ Clock fold_decision(const D& d, int last, long long owed)
{
    Clock* c = d.clk;
    ClockAux* aux = clock_aux(c);
    Clock prev = last == 0 ? *c : aux->shadow[last & 1];
    if (last == 0) prev.target += owed;
    unsigned long long* sb;
    unsigned int* fl;
    cfl_slot(c, last % 3, sb, fl);
    const Clock h = control_next(prev, *sb, *fl, d.fixed_dt, d.cfl_target, d.cfl_max, d.max_retries, 2);
    aux->slot[0].smax_bits = 0ull;
    aux->slot[0].flags = 0u;
    aux->slot[1].smax_bits = 0ull;
    aux->slot[1].flags = 0u;
    return h;
}

// Recorder: after an attempt, the running maximum of rho' along one grid row,
// kept per column of the path the (possibly moving) domain covers, and rho'
// and t at one probe column after every accepted step.  Idempotent: after a
// rejected or empty attempt it sees the state and step count it saw before,
// so it can follow every attempt without knowing which were accepted.
struct RecDesc {
    int on;                     // 0: no recorder
    int row, probe_col;
    long long path_len, base, capacity;
    double* row_max;
    double* probe_t;
    double* probe_rho;
    double rho0, t_unit;
};

// By one block of n threads: record the state that clock state h describes.
template <typename S, typename T>
__device__ __forceinline__ void record_row(const SimDesc& d, const RecDesc& r, const Clock& h, int n)
{
    const long long k = h.accepted - r.base - 1;        // index of the latest accepted step
    if (k < 0) return;
    const S* R = (const S*)d.buf[h.cur] + (size_t)r.row * d.pitch;
    for (int i = threadIdx.x; i < d.nx; i += n) {
        const double rho = (double)Codec<S, T>::ld(R[i], d.scale[0]) * r.rho0;
        const long long pc = h.x_off + i;
        if (pc < r.path_len) r.row_max[pc] = fmax(r.row_max[pc], rho);
        if (pc == r.probe_col && k < r.capacity) {
            r.probe_t[k] = h.t * r.t_unit;
            r.probe_rho[k] = rho;
        }
    }
}

// With a recorder the grid has one block more than its tiles need: the last
// one records the state the decision on the attempt before this one left (its
// buffer is the one this attempt reads), beside the tiles instead of in a
// launch of its own after every attempt (7.6 us each).  The closing launch
// records after the run's last attempt.
template <typename S, typename T>
__device__ __forceinline__ bool record_block(const SimDesc& d, const RecDesc& r, int pos, long long owed)
{
    if (!r.on || blockIdx.x != gridDim.x - 1) return false;
    if (pos >= 1) record_row<S, T>(d, r, step_clock(d, pos, owed), blockDim.x);
    return true;
}

template <typename S, typename T, int AXI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Occupancy<T>::waves)))
void k_step(SimDesc d, RecDesc r, int force, int pos, long long owed)
{
    pos = max(pos, 0);
    if (record_block<S, T>(d, r, pos, owed)) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = xcd_block(blockIdx.x, gridDim.x - r.on) * WAVES_PER_BLOCK + wave;
    if (tile >= d.strips * d.segs) return;
    Attempt at;
    if (step_begin(d, force, pos, owed, at)) march_tile<S, T, AXI>(d, tile % d.strips, tile / d.strips, at);
    if (tile == 0 && (threadIdx.x & (WAVE - 1)) == 0) step_end(d, pos, owed);
}

// The same attempt over block tiles (one block per tile): small grids, where
// march_tile would leave most of the chip idle (see block_march).  Whether a
// step is owed is the same for the whole block: every wavefront decides from
// the same words.
template <typename S, typename T, int AXI>
__global__ __launch_bounds__(WAVE * BLOCK_ROWS) __attribute__((amdgpu_waves_per_eu(4)))
void k_step_block(SimDesc d, RecDesc r, int force, int pos, long long owed)
{
    __shared__ BlockShare<T> sh;
    pos = max(pos, 0);
    if (record_block<S, T>(d, r, pos, owed)) return;
    const int tile = xcd_block(blockIdx.x, gridDim.x - r.on);
    block_tile<S, T, AXI>(d, tile % d.strips, tile / d.strips, d.block_rows, sh,
                          [&](Attempt& at) { return step_begin(d, force, pos, owed, at); });
    if (tile == 0 && threadIdx.x == 0) step_end(d, pos, owed);
}

struct TileRef { int sim, strip, seg, pad; };

// One attempted step of every simulation of a batch; each tile takes its own
// simulation's decision as k_step does, and a simulation's first tile closes it.
template <typename S, typename T, int AXI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Occupancy<T>::waves)))
void k_step_batch(const SimDesc* __restrict__ descs, const TileRef* __restrict__ tiles, int ntiles, int force, int pos,
                  long long owed)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = xcd_block(blockIdx.x, gridDim.x) * WAVES_PER_BLOCK + wave;
    if (tile >= ntiles) return;
    pos = max(pos, 0);
    const TileRef tr = tiles[tile];
    const SimDesc& d = descs[tr.sim];
    Attempt at;
    if (step_begin(d, force, pos, owed, at)) march_tile<S, T, AXI>(d, tr.strip, tr.seg, at);
    if (tr.strip == 0 && tr.seg == 0 && (threadIdx.x & (WAVE - 1)) == 0) step_end(d, pos, owed);
}

}  // namespace fvna
