// Device helpers shared by the step kernels (kernels.hip) and the adjoint
// kernels (adjoint.hip).
#pragma once
#include <hip/hip_runtime.h>
#include "common.hpp"

namespace ugk {

// The launches of step n carry K.gate = n and may be enqueued behind steps
// that have not run yet.  A launch from before the step's commit runs only
// when n steps have committed (after = 0), one from after it only when n + 1
// have (after = 1).  Behind a step that did not commit, every later step's
// launches therefore return at once and leave that step's state as its
// failure left it.  The value read is uniform, so whole grids return together.
// s = c sigma dt / eps^2 of a slot from its opacity, in one evaluation order:
// the coefficient tables store it and the sweeps re-form it from sigma alone
// (the same bits), so that they need not read both.
__device__ inline double s_of_sigma(const Consts& K, double sg) { return K.lam_scale * sg; }

__device__ inline bool gate_open(const Dev& D, const Consts& K, uint32_t after)
{
    return K.gate == GATE_OFF || *D.step == K.gate + after;
}

// The kernels of a small step are chains of waits a few hundred cycles long: on the
// arguments (over a kilobyte, 64 bytes to a line of the scalar cache, fetched line by
// line as the code reaches them) and on single words that the launch before wrote.
// warm_args touches every line of the first BYTES of the arguments at once, so that one
// wait covers them all.
template <int BYTES>
__device__ inline void warm_args()
{
#ifdef __HIP_DEVICE_COMPILE__
    const auto* p = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < BYTES; i += 64) x |= p[i / 4];
    asm volatile("" ::"s"(x));
#endif
}

// A zero the compiler does not know, one per lane: a uniform word read at p + lane_zero()
// is a vector load, which is in flight beside the slot's own loads; a scalar load of it
// would be waited for together with every argument read after it.
__device__ inline int lane_zero()
{
    int z = 0;
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(z));
#endif
    return z;
}

struct Slot {
    int inst, lcell, g;
    bool cell_ok, active;
};

// Slot j of a thread whose wavefront covers the 64 slots j & ~63 .. (j & ~63) + 63.
// Instance blocks start on multiples of 64, so those slots belong to one
// instance: it is looked up once per wavefront and its record is read with
// scalar loads.
__device__ inline Slot decode_slot(const Dev& D, const Consts& K, int64_t j)
{
    Slot s;
    const bool in = j < K.n_cg;
    const int w = __builtin_amdgcn_readfirstlane((int)(j >> 6));
    s.inst = ((int64_t)w << 6) < K.n_cg ? D.wave_inst[w] : K.n_inst - 1;
    const Inst& I = D.inst[s.inst];
    const int64_t local = j - I.cg_off;
    s.lcell = (int)(local >> I.lgGp);
    s.g = (int)(local & (I.Gp - 1));
    s.cell_ok = in && local >= 0 && s.lcell < I.ncell;
    s.active = s.cell_ok && s.g < I.G;
    return s;
}

// decode_slot, also handing out the slot's instance record: SINGLE (a context
// of one instance) takes it from the kernel arguments, with no memory read on
// the critical path; otherwise it comes from the instance table.
template <bool SINGLE>
__device__ inline Slot decode_slot_rec(const Dev& D, const Consts& K, int64_t j, Inst& I)
{
    Slot s;
    const bool in = j < K.n_cg;
    if (SINGLE) {
        s.inst = 0;
        I = K.inst0;
    } else {
        const int w = __builtin_amdgcn_readfirstlane((int)(j >> 6));
        s.inst = ((int64_t)w << 6) < K.n_cg ? D.wave_inst[w] : K.n_inst - 1;
        I = D.inst[s.inst];
    }
    const int64_t local = j - I.cg_off;
    s.lcell = (int)(local >> I.lgGp);
    s.g = (int)(local & (I.Gp - 1));
    s.cell_ok = in && local >= 0 && s.lcell < I.ncell;
    s.active = s.cell_ok && s.g < I.G;
    return s;
}

__device__ inline unsigned long long dbits(double v) { return (unsigned long long)__double_as_longlong(v); }
__device__ inline double bitsd(unsigned long long v) { return __longlong_as_double((long long)v); }


// The larger of two non-negative doubles, NaN above everything (the order of their bits).
__device__ inline double nan_max(double a, double b) { return bitsd(max(dbits(a), dbits(b))); }

// Largest value over the wavefront by DPP row steps: within quads, half rows,
// rows, then across rows (row broadcasts 15 and 31); lane 63 ends with the
// maximum, which is returned to every lane.
__device__ inline uint32_t wave_max_u32(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row_mirror
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));  // row_bcast15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));  // row_bcast31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// A double moved across lanes by one DPP step; lanes of rows outside ROW_MASK,
// and lanes whose source is outside the row, read 0.0.
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_f64(double v)
{
    const long long b = __double_as_longlong(v);
    int lo, hi;
    if (ROW_MASK == 0xF) {
        // every lane is written: no old value to set up
        lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
        hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROW_MASK, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xF, false);
    }
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// The value of the next lane (0 in lane 63), by a wavefront shift.
__device__ inline double next_lane(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x130, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x130, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// v + (v of the lane 16 or 32 lanes across) by row and half swaps of registers:
// the same sum, with the same bits, in both lanes, without the shuffles' trip
// through the LDS unit.
template <int N>
__device__ inline double add_across(double v)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
    const auto l = N == 16 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                           : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = N == 16 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                           : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    const double a = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0]));
    const double c = __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    return a + c;
}

// Sum over aligned groups of n lanes (n a power of two up to 64, the same in
// every lane).  Each step adds two partial sums that every lane of a group
// holds with the same bits, so all lanes of a group end with the same bits:
// pairs and quads (quad permutes), 8 and 16 lanes (half-row and row mirrors),
// then 32 and 64 lanes by row and half swaps.
__device__ inline double group_sum(double v, int n)
{
    if (n > 1) v += dpp_f64<0xB1, 0xF>(v);     // quad_perm 1,0,3,2
    if (n > 2) v += dpp_f64<0x4E, 0xF>(v);     // quad_perm 2,3,0,1
    if (n > 4) v += dpp_f64<0x141, 0xF>(v);    // row_half_mirror
    if (n > 8) v += dpp_f64<0x140, 0xF>(v);    // row_mirror
    if (n > 16) v = add_across<16>(v);
    if (n > 32) v = add_across<32>(v);
    return v;
}

// Sum over the wavefront, returned to every lane: the group steps up to rows,
// then the row broadcasts 15 and 31 gather the four row sums into lane 63.
__device__ inline double wave_sum(double v)
{
    v += dpp_f64<0xB1, 0xF>(v);
    v += dpp_f64<0x4E, 0xF>(v);
    v += dpp_f64<0x141, 0xF>(v);
    v += dpp_f64<0x140, 0xF>(v);
    v += dpp_f64<0x142, 0xA>(v);               // row_bcast15 into rows 1, 3
    v += dpp_f64<0x143, 0xC>(v);               // row_bcast31 into rows 2, 3
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Largest of non-negative doubles (NaN allowed) over the wavefront, as IEEE bit
// patterns: for these the unsigned order of the bits is the numeric order, and
// every NaN lies above +inf, so a NaN anywhere wins.  The high words are
// reduced first, then the low words of the lanes that hold the largest high word.
__device__ inline unsigned long long wave_max_bits(double x)
{
    const unsigned long long b = dbits(x);
    const uint32_t hi = wave_max_u32((uint32_t)(b >> 32));
    const uint32_t lo = wave_max_u32((uint32_t)(b >> 32) == hi ? (uint32_t)b : 0u);
    return ((unsigned long long)hi << 32) | lo;
}

// Block b of n works on item xcd_band(b, n): blocks go to the 8 XCDs in turn, and this
// gives each a contiguous run of items, whose neighbours its L2 then holds (sweeps of
// 256 x 256 cells of 32 groups: 230 -> 222 us a step; 285 x 285 of 24: 1371 -> 1332).
__device__ inline uint32_t xcd_band(uint32_t b, uint32_t n)
{
    const uint32_t x = b & 7u, q = n >> 3, r = n & 7u;
    return x * q + min(x, r) + (b >> 3);
}

}  // namespace ugk
