// PPM shear kernel.  Persistent: each wavefront repeatedly takes the next
// (pencil, velocity block) work item from the list built by the planner and
// marches along the pencil, one lane per velocity cell of the block (64 lanes
// = 4x4x4 cells), with the reconstruction state in registers:
//   slope of cell t-1      (Colella & Woodward 1984, eq. 1.7-1.8)
//   face value t-3/2       (eq. 1.6, uniform grid)
//   limited profile t-2    (eq. 1.10)
//   flux through t-5/2     (eq. 1.12; upwind cell chosen by the sign of the
//                           lane's Courant number)
//   new average of t-3  =  old average + F(t-7/2) - F(t-5/2), written in place.
// Each (cell, block) belongs to exactly one item of a shear, so the update is
// in place without a second buffer.  Cells that do not hold the block read as
// zero; blocks created by the planner's growth step read as zero too.
//
// Storage variants:
//   VL_F64 : everything in FP64.
//   VL_F32 / VL_BF16 : values are loaded into FP32; slopes, faces and the
//            limiter run in FP32; the Courant number, flux integral and update
//            in FP64.  The FP64 update of a cell takes the rounding residual
//            carried along the pencil (of either sign) if it holds at least
//            that much, else the carry passes it by unchanged, so no cell is
//            driven negative and positive and negative carries are treated
//            alike; the sum is rounded to the storage type and the difference
//            carried on.  A line's carry starts from the residual its last
//            shear along the same axis left for the block (its sum over the
//            block's 64 velocity cells, kept in FP64 in the axis's ledger
//            store and spread evenly over the lanes) and its final carry,
//            summed over the lanes in a fixed order, is stored there for the
//            next one, so residuals are put back into f rather than
//            accumulating.  The line's stored mass changes only by its final
//            carry minus its starting one, which the item leaves for the FP64
//            mass ledger.
#include <algorithm>

#include "vl_internal.h"
#include "vl_storage.h"

namespace vl {

struct SweepParams {
    int d, sidx, L, WL;
    int wrap;                // 0, or the period: the line's cells [H, H + wrap) are its own
                             // neighbours, seen again before and after them
    double dt;
    double sparse_min;
    const double *lg_old;    // residuals of the last shear along d, per old item
    double *lg_new;          // this shear's, per item
    const int32_t *lg_src;   // per item: its old item or -1
    int64_t lg_cap;          // items of a ledger store (0: no ledger)
};

__device__ inline void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr uint32_t ABSENT = 0xffffffffu;

// the wavefront's place-th block for the old values of a periodic line's
// first cells (the grid holds at most NSINK wavefronts)
__device__ __forceinline__ uint32_t wrap_slot(const Dev &D, int place)
{
    // (visibly uniform, so the blocks' resources are formed in scalar registers)
    const uint32_t wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return (uint32_t)D.trash + 1 + NSINK + wave * (2 * WRAP) + (uint32_t)place;
}

// The ghost cells of a periodic line in its slot table (the local cells' are
// in place): those before the line are its last cells, read where they lie,
// for the march has read them before it writes its first cell; those after
// the line are its first cells, which the march has overwritten by then, so
// their old values are copied aside first (three blocks, which stay in the
// cache; place: 0 or WRAP), so that the marches need no test for the line's
// end.  A block created in this shear is not held by the images yet.
template <int ST>
__device__ __forceinline__ void wrap_slots(const Dev &D, uint32_t *srow, int L, int n, int lane, int place)
{
    const uint32_t lane_off = (uint32_t)lane * Storage<ST>::BYTES;
    uint32_t sl[WRAP];
    typename Storage<ST>::T v[WRAP];
#pragma unroll
    for (int k = 0; k < WRAP; k++) sl[k] = __builtin_amdgcn_readfirstlane(srow[H + k]);
    const uint32_t last = srow[n + (lane < WRAP ? lane : 0)];
#pragma unroll
    for (int k = 0; k < WRAP; k++)
        if (!(sl[k] & NEWFLAG)) v[k] = block_load_raw<ST>(block_rsrc<ST>(D.pool, sl[k]), lane_off);
    if (lane < WRAP) srow[lane] = (last & NEWFLAG) ? ABSENT : last;
#pragma unroll
    for (int k = 0; k < WRAP; k++) {
        const uint32_t to = wrap_slot(D, place + k);
        if (!(sl[k] & NEWFLAG)) block_store(block_rsrc<ST>(D.pool, to), lane_off, v[k]);
        if (lane == k) srow[L - WRAP + k] = (sl[k] & NEWFLAG) ? ABSENT : to;
    }
}
constexpr int PF = 8;  // cells prefetched ahead of the reconstruction front
// A march's slot window: 64 cells from WIN0 before the front, moved on every
// WSTEP cells (so it holds the cells up to 64 - WIN0 - WSTEP ahead)
constexpr int WIN0 = 4, WSTEP = 32;
// slot table of a line: WIN0 cells before it, NM * 64 for it, and what the
// windows, the prefetches and the unconditional march's groups read beyond it
template <int NM>
constexpr int TABLE = WIN0 + 64 * NM + 72;

__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }


// a read-only array (or one whose element is read before this kernel writes
// it) read at a wave-uniform place through the scalar cache
template <typename T>
__device__ __forceinline__ T scalar_load(const T *p, int64_t i)
{
    return ((const __attribute__((address_space(4))) T *)(uintptr_t)p)[i];
}

// The residual that the last shear along the axis left for the line and block
// of an item, given the old ledger item (src < 0: the block was not on the
// line then).  Each velocity cell's carry starts from 1/64 of it; the 64 equal
// shares add up to the residual exactly.
template <int ST>
__device__ __forceinline__ double take_residual(const SweepParams &sp, int32_t src)
{
    double r = 0.0;
    if constexpr (ST != VL_F64)
        if (src >= 0) r = scalar_load(sp.lg_old, src);
    return r;
}

// Leave the line's final carry, summed over the lanes in a fixed order, for
// the next shear along the axis, and its change (final minus starting) for
// the mass ledger.
template <int ST>
__device__ __forceinline__ void leave_residual(const Dev &D, const SweepParams &sp, int64_t it, int lane,
                                               double carry, double start_sum)
{
    if constexpr (ST != VL_F64) {
        const double s = wave_sum_f64(carry);
        if (lane == 0) {
            if (it < sp.lg_cap) sp.lg_new[it] = s;
            D.resid[it] = s - start_sum;
        }
    }
}

// max(0, min(x, y)); in FP32 one median-of-three instruction (x >= 0 here,
// and a zero result takes the sign of the side afterwards, so the sign of a
// zero makes no difference)
template <typename C>
__device__ __forceinline__ C clamp_min0(C x, C y)
{
    if constexpr (std::is_same<C, float>::value)
        return __builtin_amdgcn_fmed3f(0.0f, x, y);
    else
        return fmax((C)0, fmin(x, y));
}

// twice the limited slope of a cell (CW84 eq. 1.7-1.8) from its one-sided
// differences dl, dr and the full difference d2 = a+ - a-: d2 limited to four
// times either one-sided difference, zero at an extremum.  In FP32 it is
// minmod(d2, minmod(4 dl, 4 dr)) with minmod(x, y) = median(x, y, 0) (the
// smaller magnitude when x and y share a sign, else zero): two median-of-three
// instructions, the same value as the general form (which FP64 keeps) up to
// the sign of a zero.  Doubled, as the half of d2 would be rounded where it is
// below the smallest normal number (the tails of a cold plasma in FP32), and
// all variants have to agree there as well.
template <typename C>
__device__ __forceinline__ C limited_slope2(C dl, C dr, C d2)
{
    if constexpr (std::is_same<C, float>::value) {
        return __builtin_amdgcn_fmed3f(d2, __builtin_amdgcn_fmed3f(4.0f * dl, 4.0f * dr, 0.0f), 0.0f);
    } else {
        const C s4 = copysign((C)4.0, d2);
        const C m = fmax((C)0, fmin(fmin(fabs(d2), s4 * dl), s4 * dr));
        return copysign(m, d2);
    }
}

// the face between a cell of average a0 and the next, d above it, with twice
// their limited slopes s0 and s1 (CW84 eq. 1.6; the fused operations written
// out, as a march's start, its iterations and all variants have to agree to the
// last bit)
__device__ __forceinline__ float face_value(float a0, float d, float s1, float s0)
{
    return fmaf(-(s1 - s0), (float)(0.5 / 6.0), fmaf(0.5f, d, a0));
}
__device__ __forceinline__ double face_value(double a0, double d, double s1, double s0)
{
    return fma(-(s1 - s0), 0.5 / 6.0, fma(0.5, d, a0));
}

// the monotonicity limiter's face offset x given the other side's offset y
// (CW84 eq. 1.10 written on the offsets): x limited to twice y, zero unless
// they share a sign (the extremum case); in FP32 minmod(x, 2 y), one
// median-of-three instruction
template <typename C>
__device__ __forceinline__ C limited_offset(C x, C y)
{
    if constexpr (std::is_same<C, float>::value)
        return __builtin_amdgcn_fmed3f(x, 2.0f * y, 0.0f);
    else
        return copysign(clamp_min0(fabs(x), copysign((C)2.0, x) * y), x);
}

// The FP64 update x of a cell (its carry included) in the storage type (a
// negative sum, which only FP32 reconstruction rounding can leave, is stored
// as zero).  nv receives the stored value in FP64, so the caller carries
// x - nv on, which keeps the pencil's mass exact whatever the rounding.  BF16: FP64 -> FP32 to nearest, then FP32 -> BF16 to nearest
// even by the hardware conversion (two roundings; they differ from one
// correct rounding only where the FP32 value lands on a BF16 midpoint).
__device__ __forceinline__ float narrow_f32(double x, double &nv)
{
    const float q = fmaxf((float)x, 0.0f);
    nv = (double)q;
    return q;
}
__device__ __forceinline__ uint16_t narrow_bf16(double x, double &nv)
{
    float t = fmaxf((float)x, 0.0f);
    __asm__("" : "+v"(t));  // keeps the two roundings apart (no fused FP64 -> BF16 rounding)
    const uint16_t h = __builtin_bit_cast(uint16_t, (__bf16)t);
    nv = (double)bf16_to_f32(h);
    return h;
}

// Blocks are read and written through buffer resources made in scalar
// registers (block_rsrc, block_load, block_store), so no vector instruction
// computes addresses in the marches.

// One (pencil, block) item: march along the pencil.  DIR = +1 when every
// lane's Courant number is positive, -1 when every one is negative, 0 when
// the block straddles v = 0 (then the upwind side is chosen per lane).
//
// The reconstruction is Colella & Woodward's, written in forms with fewer
// operations that give the same values:
//  * twice the limited slope: copysign(max(0, min(|c|, 4 s dl, 4 s dr)), c)
//    with c = a+ - a- and s = sign(c) (zero unless dl and dr share a sign),
//    in FP32 minmod(c, minmod(4 dl, 4 dr)) (limited_slope2), the faces'
//    factor 1/6 halved;
//  * monotonicity limiter on the face offsets dL = a - aL, dR = aR - a: the
//    two overshoot corrections of the limiter are dL' = min(|dL|, 2|dR|) and
//    dR' = min(|dR|, 2|dL|) (with the sign of the side), the extremum case is
//    dL' = dR' = 0;
//  * flux integral of the parabola over the upwind fraction |c| of the cell,
//    expanded in dL', dR': F = c a + P dR' + Q dL' with
//    P = c (1-c)^2, Q = c^2 (1-c) for c > 0 and P = s^2 (1-s), Q = s (1-s)^2
//    for c = -s < 0.
// Variant "unconditional stores": slots of 8 cells at a time from LDS into
// scalar registers; every iteration stores (to a per-wavefront sink block when
// there is nothing to write), which keeps the compiler's memory counters exact.
template <int ST, int DIR, bool LAST>
__device__ __forceinline__ void march_unc(const Dev &D, const uint32_t *srow, uint8_t *sflag, int L, double c,
                                          int lane, double smin, double &carry, int tb, int te)
{
    using C = typename std::conditional<ST == VL_F64, double, float>::type;  // reconstruction type
    const bool pos = (DIR > 0) ? true : (DIR < 0) ? false : (c > 0.0);
    const double s = fabs(c);
    const double P = pos ? c * (1.0 - c) * (1.0 - c) : s * s * (1.0 - s);
    const double Q = pos ? c * c * (1.0 - c) : s * (1.0 - s) * (1.0 - s);
    constexpr int BS = Storage<ST>::BYTES;
    const uint32_t lane_off = (uint32_t)lane * BS;
    const uint32_t zslot = (uint32_t)D.trash;     // all-zero block: reads of absent cells
    // write-only block for discarded stores, one per wavefront
    const uint32_t sink = (uint32_t)D.trash + 1 +
                          (uint32_t)((blockIdx.x * 4 + (threadIdx.x >> 6)) % NSINK);

    // slots of 8 consecutive cells (raw: slot, slot|NEWFLAG or ABSENT), wave-uniform
    auto slots8 = [&](int t, uint32_t (&o)[PF]) {
        const uint4 v0 = *(const uint4 *)(srow + t);
        const uint4 v1 = *(const uint4 *)(srow + t + 4);
        o[0] = uniform_u32(v0.x); o[1] = uniform_u32(v0.y); o[2] = uniform_u32(v0.z); o[3] = uniform_u32(v0.w);
        o[4] = uniform_u32(v1.x); o[5] = uniform_u32(v1.y); o[6] = uniform_u32(v1.z); o[7] = uniform_u32(v1.w);
    };
    auto fetch = [&](uint32_t raw) -> C {
        const uint32_t sl = (raw & NEWFLAG) ? zslot : raw;  // absent or created this shear: zero
        const char *blk = (const char *)D.pool + (uint64_t)sl * (BLK * BS);
        if constexpr (ST == VL_F64)
            return *(const double *)(blk + lane_off);
        else if constexpr (ST == VL_F32)
            return *(const float *)(blk + lane_off);
        else
            return bf16_to_f32(*(const uint16_t *)(blk + lane_off));
    };

    C a1 = 0, a2 = 0;           // a(t-1), a(t-2)
    double a3d = 0.0;           // a(t-3) in FP64 (last iteration's a(t-2))
    C da_prev = 0;              // slope of cell t-2
    C face_prev = 0;            // face t-5/2
    double Fc_prev = 0.0, Ff_prev = 0.0;
    uint32_t prv[PF], cur[PF], nxt[PF];
    C q[PF];
#pragma unroll
    for (int u = 0; u < PF; u++) prv[u] = ABSENT;
    const int t00 = tb & ~3;  // the slot table is read in aligned groups of 4
    slots8(t00, cur);
#pragma unroll
    for (int u = 0; u < PF; u++) q[u] = fetch(cur[u]);
    for (int t0 = t00; t0 < te; t0 += PF) {
        slots8(t0 + PF, nxt);
#pragma unroll
        for (int u = 0; u < PF; u++) {
            const int t = t0 + u;
            const C a = q[u];
            q[u] = fetch(nxt[u]);
            // slope of cell t-1
            const C dl = a1 - a2, dr = a - a1;
            const C da = limited_slope2(dl, dr, a - a2);
            // face between t-2 and t-1
            const C face = face_value(a2, a1 - a2, da, da_prev);
            // limited face offsets of cell t-2
            const C ai = a2;
            const C dL = ai - face_prev, dR = face - ai;
            const double dLp = (double)limited_offset(dL, dR), dRp = (double)limited_offset(dR, dL);
            const double aid = (double)ai;
            const double Fc = fma(P, dRp, fma(Q, dLp, c * aid));
            const double Ff = (DIR > 0) ? Fc_prev : (DIR < 0) ? Fc : (pos ? Fc_prev : Fc);
            // new value of cell t-3, stored unconditionally (to the sink when
            // there is nothing to store) so the memory counters stay exact
            const uint32_t raw3 = (u >= 3) ? cur[u - 3] : prv[u + PF - 3];
            // the march runs in whole groups past te; cells from there on
            // belong to the next segment and are written by its own march
            const bool live = (t >= 6) && (t < L) && (t < te) && (raw3 != ABSENT);
            const uint32_t s3 = live ? (raw3 & ~NEWFLAG) : sink;
            char *dst = (char *)D.pool + (uint64_t)s3 * (BLK * BS);
            double nv;
            if constexpr (ST == VL_F64) {
                nv = a3d + (Ff_prev - Ff);
                *(double *)(dst + lane_off) = nv;
            } else {
                // the carry goes into the cell only if the cell holds at least as much
                const double base = a3d + (Ff_prev - Ff);
                const double cin = (live && fabs(carry) <= base) ? carry : 0.0;
                const double x = base + cin;
                if constexpr (ST == VL_F32)
                    *(float *)(dst + lane_off) = narrow_f32(x, nv);
                else
                    *(uint16_t *)(dst + lane_off) = narrow_bf16(x, nv);
                if (live) carry = (carry - cin) + (x - nv);
            }
            if constexpr (LAST) {
                const unsigned long long any = __ballot(nv >= smin);
                if (t >= 3 && t < te) sflag[t - 3] = any ? 1 : 0;  // same value from every lane
            }
            a3d = aid;
            a2 = a1;
            a1 = a;
            da_prev = da;
            face_prev = face;
            Fc_prev = Fc;
            Ff_prev = Ff;
        }
#pragma unroll
        for (int u = 0; u < PF; u++) {
            prv[u] = cur[u];
            cur[u] = nxt[u];
        }
    }
}


// Variant "conditional stores": 64 cells' slots at a time lie one per lane in
// a window register (reread from the LDS table every 32 cells), a cell's slot
// is broadcast from its lane when the cell is fetched (prefetch distance PFV)
// and kept in scalar registers until the cell is written PFV + 3 iterations
// later.  A cell without the block, or with one created this shear, is read
// through a resource of no records: the hardware returns zero and moves
// nothing.  The window's cells to be written are one scalar mask, so a store
// costs one bit test (scalar branch).
template <int ST, int DIR, bool LAST, int PFV>
__device__ __forceinline__ void march_cond(const Dev &D, const uint32_t *srow, uint8_t *sflag, int L, double c,
                                           int lane, double smin, double &carry, int tb, int te)
{
    static_assert(PFV >= 3 && PFV <= 16, "the written cell's slot comes from the previous group; window of 64 cells");
    using C = typename std::conditional<ST == VL_F64, double, float>::type;  // reconstruction type
    const bool pos = (DIR > 0) ? true : (DIR < 0) ? false : (c > 0.0);
    const double s = fabs(c);
    const double P = pos ? c * (1.0 - c) * (1.0 - c) : s * s * (1.0 - s);
    const double Q = pos ? c * c * (1.0 - c) : s * (1.0 - s) * (1.0 - s);
    constexpr int BS = Storage<ST>::BYTES;
    const uint32_t lane_off = (uint32_t)lane * BS;

    // a cell's value from its raw slot (wave-uniform); flagged slots: zero
    auto fetch_raw = [&](uint32_t sl) -> C {
        return block_load<ST>(block_rsrc_if<ST>(D.pool, sl, (int32_t)sl >= 0), lane_off);
    };

    // The front starts at cell tb + 2: with zeros before cell tb, the fluxes
    // of the cells before it are zero, and the state at tb + 2 is the slope of
    // cell tb and the face below it.  It ends with the cell te - 1, whose
    // iteration writes the segment's last cell (a check per iteration: runs of
    // nine cells, usual on the lines of a mixture's hot blobs, take 10
    // iterations instead of 12 to 16 in whole groups from tb).
    const int t_first = tb + 2;
    C q[PFV];
    // raw slots of the cells t0 .. t0+PFV-1 (fetched by the previous group or
    // the prologue), of the three cells before them, and of the cells this
    // group fetches
    uint32_t prv[PFV], bef[3], cur[PFV];
    // lane j of the window holds cell w0 - WIN0 + j
    uint32_t win = srow[t_first - WIN0 + lane];
#pragma unroll
    for (int i = 0; i < 3; i++) bef[i] = (uint32_t)__builtin_amdgcn_readlane((int)win, WIN0 - 3 + i);
    C a2 = fetch_raw(bef[1]), a1 = fetch_raw(bef[2]);  // cells t-2, t-1
#pragma unroll
    for (int u = 0; u < PFV; u++) {
        prv[u] = (uint32_t)__builtin_amdgcn_readlane((int)win, WIN0 + u);
        q[u] = fetch_raw(prv[u]);
    }
    double a3d = 0.0;
    C da_prev = limited_slope2(a2, a1 - a2, a1);
    C face_prev = face_value((C)0, a2, da_prev, (C)0);
    double Fc_prev = 0.0, Ff_prev = 0.0;
    for (int w0 = t_first; w0 < te; w0 += WSTEP) {
        if (w0 != t_first) win = srow[w0 - WIN0 + lane];
        // the window's cells that this march writes: local ones before te - 3
        // (those from there on belong to the next segment's march)
        const int jlo = max(0, H + WIN0 - w0), jhi = min(L - H, te - 3) + WIN0 - w0;
        unsigned long long wm = __ballot(win != ABSENT && lane >= jlo && lane < jhi) >> (WIN0 - 3);
        const int iend = min(WSTEP, te - w0);
        // one iteration, cell t = w0 + i0 + u; slot3 is the slot of cell t - 3
        auto iteration = [&](C a, uint32_t slot3, bool write, int t) {
            const C dl = a1 - a2, dr = a - a1;
            const C da = limited_slope2(dl, dr, a - a2);
            const C face = face_value(a2, a1 - a2, da, da_prev);
            const C ai = a2;
            const C dL = ai - face_prev, dR = face - ai;
            const double dLp = (double)limited_offset(dL, dR), dRp = (double)limited_offset(dR, dL);
            const double aid = (double)ai;
            const double Fc = fma(P, dRp, fma(Q, dLp, c * aid));
            const double Ff = (DIR > 0) ? Fc_prev : (DIR < 0) ? Fc : (pos ? Fc_prev : Fc);
            if (write) {
                const __amdgpu_buffer_rsrc_t dst = block_rsrc<ST>(D.pool, slot3 & ~NEWFLAG);
                double nv;
                if constexpr (ST == VL_F64) {
                    nv = a3d + (Ff_prev - Ff);
                    block_store(dst, lane_off, nv);
                } else {
                    // the carry goes into the cell only if the cell holds at least as much
                    const double base = a3d + (Ff_prev - Ff);
                    const double cin = (fabs(carry) <= base) ? carry : 0.0;
                    const double x = base + cin;
                    if constexpr (ST == VL_F32)
                        block_store(dst, lane_off, narrow_f32(x, nv));
                    else
                        block_store(dst, lane_off, narrow_bf16(x, nv));
                    carry = (carry - cin) + (x - nv);
                }
                if constexpr (LAST) {
                    const unsigned long long any = __ballot(nv >= smin);
                    sflag[t - 3] = any ? 1 : 0;
                }
            }
            a3d = aid;
            a2 = a1;
            a1 = a;
            da_prev = da;
            face_prev = face;
            Fc_prev = Fc;
            Ff_prev = Ff;
        };
        int i0 = 0;
        for (; i0 + PFV <= iend; i0 += PFV) {
#pragma unroll
            for (int u = 0; u < PFV; u++) {
                cur[u] = (uint32_t)__builtin_amdgcn_readlane((int)win, i0 + u + PFV + WIN0);
                const C a = q[u];
                q[u] = fetch_raw(cur[u]);
                iteration(a, (u >= 3) ? prv[u - 3] : bef[u], (wm >> u) & 1ull, w0 + i0 + u);
            }
            wm >>= PFV;
#pragma unroll
            for (int i = 0; i < 3; i++) bef[i] = prv[PFV - 3 + i];
#pragma unroll
            for (int u = 0; u < PFV; u++) prv[u] = cur[u];
        }
        // the segment's last iterations, less than a group, with nothing left
        // to fetch
        if (i0 < iend) {
#pragma unroll
            for (int u = 0; u < PFV - 1; u++)
                if (i0 + u < iend)
                    iteration(q[u], (u >= 3) ? prv[u - 3] : bef[u], (wm >> u) & 1ull, w0 + i0 + u);
        }
    }
}

// shear variants chosen by the autotuner (all give bit-identical results)
//   style 0: conditional stores, style 1: unconditional stores, style 2:
//   conditional stores with the items of a wavefront streamed (the next
//   item's slot table and first cells are loaded during the current item)
//   pf: prefetch distance; minw: minimum waves per SIMD asked of the compiler (0 = default)
struct VariantInfo {
    int style, pf, minw;
};
// The first is what an untuned partition runs.  Eight waves per SIMD leave it
// 64 VGPRs, which BF16 on lines of up to 64 cells fits; the others spill a few
// per item, outside the marches' loops (lines of up to 64 / 128 / 256 cells,
// first shears and last: FP64 3, 3 / 3, 5 / 10, 14, FP32 2, 2 / 2, 4 / 4, 6,
// BF16 0, 0 / 1, 3 / 3, 3).  ms per 1e9 cells read and written, the three shears
// together, variants 0 : 8 : 7 : 1 : 3 (2 and 10 behind 7 everywhere but on 8^3
// cells, where they lead 0 by 5 % and 3 %):
//   16x16x8 sparse FP64     6.36 : 6.66 : 6.53 : 6.70 : 6.97
//   64x64x32 sparse FP64    5.83 : 5.86 : 5.83 : 5.90 : 5.81
//   16x128x16 sparse FP64   6.15 : 6.30 : 6.18 : 6.27 : 6.50
//   8x250x8 sparse FP64     6.94 : 7.25 : 7.00 : 7.14 : 7.31
//   23x17x11 sparse FP32    4.33 : 4.07 : 4.81 : 5.19 : 4.55
//   40x40x20 mixture FP32   3.37 : 3.31 : 3.81 : 3.92 : 3.51
//   8x250x8 sparse FP32     4.76 : 4.59 : 5.11 : 5.35 : 4.96
//   24x24x12 mixture BF16   3.97 : 4.17 : 4.73 : 4.78 : 4.89
//   64x64x32 mixture BF16   3.24 : 3.33 : 3.56 : 3.61 : 3.69
//   128x128x8 mixture BF16  3.62 : 3.75 : 4.06 : 4.08 : 4.20
//   8x250x8 sparse BF16     4.14 : 4.18 : 4.67 : 4.74 : 4.81
// so beyond 8^3 cells it is the fastest or within 1 % of it in FP64 and BF16, and
// up to 6 % behind variant 8 in FP32.
constexpr VariantInfo VARIANTS[] = {{0, 4, 8}, {0, 8, 6}, {0, 4, 0}, {0, 16, 0}, {1, 8, 0}, {1, 8, 5},
                                   {2, 8, 0}, {0, 8, 0}, {0, 8, 8}, {2, 8, 8}, {0, 4, 6}};
constexpr int NVARIANTS = sizeof(VARIANTS) / sizeof(VARIANTS[0]);

template <int ST, int DIR, bool LAST, int V>
__device__ __forceinline__ void march(const Dev &D, const uint32_t *srow, uint8_t *sflag, int L, double c,
                                      int lane, double smin, double &carry, int tb, int te)
{
    constexpr VariantInfo vi = VARIANTS[V];
    if constexpr (vi.style == 1)
        march_unc<ST, DIR, LAST>(D, srow, sflag, L, c, lane, smin, carry, tb, te);
    else
        march_cond<ST, DIR, LAST, vi.pf>(D, srow, sflag, L, c, lane, smin, carry, tb, te);
}

// Content flags of the last shear for an item: bit t of word t / 32 tells
// whether local cell t of the pencil holds the block with a value >=
// sparse_min after the update.  The words replace the item's presence masks
// (read at the item's start, not needed after it) in one coalesced store; the
// pruning finds them through the item recorded for each list entry.
__device__ __forceinline__ void store_flag_words(const Dev &D, int64_t it, const uint32_t *srow,
                                                 const uint8_t *sflag, int L, int lane)
{
    uint32_t word = 0;
    for (int t0 = 0; t0 < L; t0 += 64) {
        const int t = t0 + lane;
        bool f = false;
        if (t >= H && t < L - H) {
            const uint32_t raw = srow[t];
            f = raw != ABSENT && (raw & ~NEWFLAG) < (uint32_t)D.lcap && sflag[t] != 0;
        }
        const unsigned long long b = __ballot(f);
        const int w = t0 >> 5;
        if (lane == w) word = (uint32_t)b;
        if (lane == w + 1) word = (uint32_t)(b >> 32);
    }
    if (lane < D.wlmax) D.masks[it * D.wlmax + lane] = word;
}

// lowest set bit at position >= from of an NM-word mask, or -1
template <int NM>
__device__ __forceinline__ int first_bit(const uint64_t (&v)[NM], int from)
{
#pragma unroll
    for (int w = 0; w < NM; w++) {
        const int f = from - 64 * w;
        const uint64_t x = v[w] & (f <= 0 ? ~0ull : f < 64 ? ~0ull << (f & 63) : 0ull);
        if (x) return 64 * w + __builtin_ctzll(x);
    }
    return -1;
}

template <int NM>
__device__ __forceinline__ int last_bit(const uint64_t (&v)[NM])
{
#pragma unroll
    for (int w = NM - 1; w >= 0; w--)
        if (v[w]) return 64 * w + 63 - __builtin_clzll(v[w]);
    return -1;
}

// word w of an NM-word mask moved down by s (0 < s < 64), ones coming in
template <int NM>
__device__ __forceinline__ uint64_t down(const uint64_t (&v)[NM], int w, int s)
{
    return (v[w] >> s) | ((w + 1 < NM ? v[w + 1 < NM ? w + 1 : w] : ~0ull) << (64 - s));
}

// an item's place in the row table, presence mask and old ledger item
template <int NM>
struct ItemMeta {
    int32_t bd, src;
    int64_t rowoff;
    uint64_t m[NM];
};

template <int ST, int NM>
__device__ __forceinline__ ItemMeta<NM> load_meta(const Dev &D, const SweepParams &sp, int64_t it)
{
    ItemMeta<NM> M;
    const int32_t *ip = (const int32_t *)(D.items + it);
    static_assert(sizeof(Item) == 16 && offsetof(Item, key) == 4 && offsetof(Item, rowoff) == 8, "item layout");
    M.bd = scalar_load(ip, 1);
    M.rowoff = scalar_load((const int64_t *)ip, 1);
    const uint32_t *mw = D.masks + it * D.wlmax;
#pragma unroll
    for (int w = 0; w < NM; w++) {
        // (words past the mask are not read)
        const uint32_t lo = scalar_load(mw, min(2 * w, sp.WL - 1)), hi = scalar_load(mw, min(2 * w + 1, sp.WL - 1));
        M.m[w] = (2 * w < sp.WL ? (uint64_t)lo : 0ull) | (2 * w + 1 < sp.WL ? (uint64_t)hi << 32 : 0ull);
    }
    M.src = -1;
    if constexpr (ST != VL_F64)
        if (it < sp.lg_cap) M.src = scalar_load(sp.lg_src, it);
    return M;
}

// the item's compacted row, lane l the entries l, l + 64, ..
template <int NM>
__device__ __forceinline__ void load_row(const Dev &D, const SweepParams &sp, const ItemMeta<NM> &M, int lane,
                                         uint32_t (&rv)[NM])
{
    int n = 0;
#pragma unroll
    for (int w = 0; w < NM; w++) n += __popcll(M.m[w]);
    if (sp.wrap) {  // the row holds the line's own cells
        n -= __popcll(M.m[0] & 7ull);
#pragma unroll
        for (int w = 0; w < NM; w++) {
            const int f = H + sp.wrap - 64 * w;  // first place past the line
            n -= __popcll(M.m[w] & (f <= 0 ? ~0ull : f < 64 ? ~0ull << (f & 63) : 0ull));
        }
    }
#pragma unroll
    for (int k = 0; k < NM; k++) rv[k] = lane + 64 * k < n ? (uint32_t)D.rows[M.rowoff + lane + 64 * k] : ABSENT;
}

// What an item costs beside its march (its index, mask, row and residual: a
// chain of dependent reads) is taken off the short lines' time by reading the
// next item's index, mask and residual into scalar registers and its row into
// a vector register before the current item's march, and by holding the mask
// as NM 64-bit scalar words (NM by the line's length), on which segments and
// ranks take a handful of instructions.  With eight 32-bit words for every
// length and all reads at the item's start the setup was 2/5 of the vector
// instructions of 24-cell BF16 lines (97 per updated cell, now 72), and the
// registers it held allowed five waves per SIMD where eight run now: step of
// the 24x24x12 BF16 mixture 9.7 -> 7.7 ms, 16x16x8 FP64 2.80 -> 2.36 ms.
template <int ST, bool LAST, int V, int NM>
__device__ __forceinline__ void sweep_body(const Dev &D, const SweepParams &sp)
{
    __shared__ __align__(16) uint32_t s_tab[4][TABLE<NM>];
    __shared__ uint32_t s_row[4][64 * NM];
    __shared__ uint8_t s_flag[4][64 * NM + 48];
    __shared__ uint32_t s_seg[4][64 * NM / 7 + 2];  // segments of the item: first cell | end << 16
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d = sp.d, L = sp.L;
    const int64_t nitems = min((int64_t)D.ctl->n_items[sp.sidx], D.item_cap);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    uint32_t *srow = s_tab[wv] + WIN0;
    uint32_t *sseg = s_seg[wv];
    uint8_t *sflag = s_flag[wv];

    int64_t it = (int64_t)blockIdx.x * 4 + wv;
    if (it >= nitems) return;
    // no cell before the line and past its mask words
    const int lane0 = threadIdx.x & 63;
    if (lane0 < WIN0) s_tab[wv][lane0] = ABSENT;
    for (int t = 64 * NM + lane0; t < TABLE<NM> - WIN0; t += 64) srow[t] = ABSENT;
    ItemMeta<NM> M = load_meta<ST, NM>(D, sp, it);
    uint32_t rv[NM];
    load_row<NM>(D, sp, M, lane0, rv);
    double start_sum = take_residual<ST>(sp, M.src);
    for (; it < nitems; it += nwaves) {
        // the lane's index as a value of this item (an empty asm the compiler
        // cannot see through), so per-lane index arithmetic is redone per item
        // rather than held in registers through the marches
        int lane = threadIdx.x & 63;
        __asm__ volatile("" : "+v"(lane));
        const ItemMeta<NM> N = load_meta<ST, NM>(D, sp, it + nwaves < nitems ? it + nwaves : it);
        uint64_t any = 0;
#pragma unroll
        for (int w = 0; w < NM; w++) any |= M.m[w];
        double carry = start_sum * (1.0 / BLK);
        if (any == 0) {  // empty item: no updated cell, the residual passes on
            leave_residual<ST>(D, sp, it, lane, carry, start_sum);
            load_row<NM>(D, sp, N, lane, rv);
            start_sum = take_residual<ST>(sp, N.src);
            M = N;
            continue;
        }
        // per-cell slot table of this item in LDS: slot, slot|NEWFLAG or ABSENT
        {
#pragma unroll
            for (int k = 0; k < NM; k++) s_row[wv][lane + 64 * k] = rv[k];
            wave_sync_lds();
            int base = sp.wrap ? -__popcll(M.m[0] & 7ull) : 0;
            const int c0 = sp.wrap ? H : 0, c1 = sp.wrap ? H + sp.wrap : L;
#pragma unroll
            for (int k = 0; k < NM; k++) {
                const int t = lane + 64 * k;
                const bool pr = ((M.m[k] >> lane) & 1ull) && t >= c0 && t < c1;
                const int rk = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(M.m[k] >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)M.m[k], 0));
                srow[t] = pr ? s_row[wv][rk] : ABSENT;
                base += __popcll(M.m[k]);
            }
        }
        wave_sync_lds();
        if (sp.wrap) {
            wrap_slots<ST>(D, srow, L, sp.wrap, lane, 0);
            wave_sync_lds();
        }
        // the next item's row and residual, on their way during the march
        load_row<NM>(D, sp, N, lane, rv);
        const double next_sum = take_residual<ST>(sp, N.src);

        const int ld = (d == 0) ? (lane & 3) : (d == 1) ? ((lane >> 2) & 3) : (lane >> 4);
        const double c = courant(D, d, 4 * M.bd + ld, sp.dt);
        const unsigned long long npos = __ballot(c > 0.0), nneg = __ballot(c < 0.0);
        // March each segment of cells holding the block: from its first such
        // cell to three past its last (where the last one is written).  Before
        // a segment's first cell at least 6 cells read as zero, so the
        // reconstruction state there is the zero state a march starts from;
        // the rounding carry runs on across segments.
        // The segments are listed in LDS first, so the masks need no
        // registers during the marches.
        int nseg = 0;
        {
            // starts of gaps of at least 6 cells without the block
            uint64_t z[NM], z2[NM], gap[NM];
#pragma unroll
            for (int w = 0; w < NM; w++) z[w] = ~M.m[w];
#pragma unroll
            for (int w = 0; w < NM; w++) z2[w] = z[w] & down<NM>(z, w, 1);
#pragma unroll
            for (int w = 0; w < NM; w++)
                gap[w] = z2[w] & down<NM>(z2, w, 2) & down<NM>(z2, w, 4) &
                         ((M.m[w] << 1) | (w > 0 ? M.m[w > 0 ? w - 1 : 0] >> 63 : 0ull));
            for (int tb = first_bit<NM>(M.m, 0); tb >= 0;) {
                const int g = first_bit<NM>(gap, tb + 1);
                const int te = (g >= 0) ? g + 3 : last_bit<NM>(M.m) + 4;
                if (lane == 0) sseg[nseg] = (uint32_t)tb | ((uint32_t)te << 16);
                nseg++;
                tb = (g >= 0) ? first_bit<NM>(M.m, g) : -1;
            }
        }
        wave_sync_lds();
        for (int k = 0; k < nseg; k++) {
            const uint32_t v = uniform_u32(sseg[k]);
            const int tb = (int)(v & 0xffffu), te = (int)(v >> 16);
            if (npos == ~0ull)
                march<ST, 1, LAST, V>(D, srow, sflag, L, c, lane, sp.sparse_min, carry, tb, te);
            else if (nneg == ~0ull)
                march<ST, -1, LAST, V>(D, srow, sflag, L, c, lane, sp.sparse_min, carry, tb, te);
            else
                march<ST, 0, LAST, V>(D, srow, sflag, L, c, lane, sp.sparse_min, carry, tb, te);
        }
        if constexpr (LAST) {
            wave_sync_lds();
            store_flag_words(D, it, srow, sflag, L, lane);
        }

        // the line's final carry (the ledger takes those of the local pencils)
        leave_residual<ST>(D, sp, it, lane, carry, start_sum);
        wave_sync_lds();
        M = N;
        start_sum = next_sum;
    }
}


// ---------------------------------------------------------------------------
// streamed items (style 2)
// ---------------------------------------------------------------------------
// Build the per-cell slot table of item `it` into srow[0 .. L+40) (wrap: see
// SweepParams; place: the wavefront's blocks for this table).
template <int ST>
__device__ __forceinline__ void build_slots(const Dev &D, int64_t it, int64_t nitems, int L, int WL, int wrap,
                                            int place, int lane, uint32_t *srow)
{
    if (it >= nitems) {
        for (int t = lane; t < L + 40; t += 64) srow[t] = ABSENT;
        return;
    }
    const Item item = D.items[it];
    uint32_t m[MAXWL];
    int pre[MAXWL + 1];
    pre[0] = 0;
#pragma unroll
    for (int w = 0; w < MAXWL; w++) {
        m[w] = (w < WL) ? D.masks[it * D.wlmax + w] : 0u;
        pre[w + 1] = pre[w] + __popc(m[w]);
    }
    const int c0 = wrap ? H : 0, c1 = wrap ? H + wrap : L;
    const int left = wrap ? __popc(m[0] & 7u) : 0;
    const int half = lane >> 5, b = lane & 31;
#pragma unroll
    for (int w = 0; w < MAXWL; w += 2) {
        if (w < WL) {
            const uint32_t mw = half ? m[w + 1] : m[w];
            const int base = (half ? pre[w + 1] : pre[w]) - left;
            const int t = 32 * (w + half) + b;
            if (t < L) {
                const bool pr = ((mw >> b) & 1u) && t >= c0 && t < c1;
                const int rk = base + __popc(mw & ((1u << b) - 1u));
                srow[t] = pr ? (uint32_t)D.rows[item.rowoff + rk] : ABSENT;
            }
        }
    }
    for (int t = L + lane; t < L + 40; t += 64) srow[t] = ABSENT;
    if (wrap) {
        wave_sync_lds();
        wrap_slots<ST>(D, srow, L, wrap, lane, place);
    }
}

// One item of the stream: cells of X; q holds X's first 8 values on entry and
// the next item's (table Y) first 8 on exit.  build_next() fills Y.
template <int ST, int DIR, bool LAST, typename BUILD>
__device__ __forceinline__ void march_stream(const Dev &D, const uint32_t *X, const uint32_t *Y, uint8_t *sflag,
                                             int L, double c, int lane, double smin, double &carry,
                                             typename std::conditional<ST == VL_F64, double, float>::type (&q)[8],
                                             BUILD build_next)
{
    using C = typename std::conditional<ST == VL_F64, double, float>::type;
    const bool pos = (DIR > 0) ? true : (DIR < 0) ? false : (c > 0.0);
    const double s = fabs(c);
    const double P = pos ? c * (1.0 - c) * (1.0 - c) : s * s * (1.0 - s);
    const double Q = pos ? c * c * (1.0 - c) : s * (1.0 - s) * (1.0 - s);
    constexpr int BS = Storage<ST>::BYTES;
    const uint32_t lane_off = (uint32_t)lane * BS;
    const uint32_t zslot = (uint32_t)D.trash;
    auto fetch = [&](const uint32_t *tab, int t) -> C {
        uint32_t sl = uniform_u32(tab[t]);
        sl = (sl & NEWFLAG) ? zslot : sl;
        const char *blk = (const char *)D.pool + (uint64_t)sl * (BLK * BS);
        if constexpr (ST == VL_F64)
            return *(const double *)(blk + lane_off);
        else if constexpr (ST == VL_F32)
            return *(const float *)(blk + lane_off);
        else
            return bf16_to_f32(*(const uint16_t *)(blk + lane_off));
    };
    C a1 = 0, a2 = 0, da_prev = 0, face_prev = 0;
    double a3d = 0.0, Fc_prev = 0.0, Ff_prev = 0.0;
    const int G = (L + 7) / 8;
    if (G == 1) build_next();
    for (int g = 0; g < G; g++) {
        const bool lastg = (g == G - 1);
        const uint32_t *src = lastg ? Y : X;
        const int fb = lastg ? 0 : 8 * (g + 1);
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int t = 8 * g + u;
            const C a = q[u];
            q[u] = fetch(src, fb + u);
            const C dl = a1 - a2, dr = a - a1;
            const C da = limited_slope2(dl, dr, a - a2);
            const C face = face_value(a2, dl, da, da_prev);
            const C ai = a2;
            const C dL = ai - face_prev, dR = face - ai;
            const double dLp = (double)limited_offset(dL, dR), dRp = (double)limited_offset(dR, dL);
            const double aid = (double)ai;
            const double Fc = fma(P, dRp, fma(Q, dLp, c * aid));
            const double Ff = (DIR > 0) ? Fc_prev : (DIR < 0) ? Fc : (pos ? Fc_prev : Fc);
            if (t >= 6 && t < L) {
                const uint32_t sl3 = uniform_u32(X[t - 3]);
                if (sl3 != ABSENT) {
                    const uint32_t s3 = sl3 & ~NEWFLAG;
                    char *dst = (char *)D.pool + (uint64_t)s3 * (BLK * BS);
                    double nv;
                    if constexpr (ST == VL_F64) {
                        nv = a3d + (Ff_prev - Ff);
                        *(double *)(dst + lane_off) = nv;
                    } else {
                        const double base = a3d + (Ff_prev - Ff);
                        const double cin = (fabs(carry) <= base) ? carry : 0.0;
                        const double x = base + cin;
                        if constexpr (ST == VL_F32)
                            *(float *)(dst + lane_off) = narrow_f32(x, nv);
                        else
                            *(uint16_t *)(dst + lane_off) = narrow_bf16(x, nv);
                        carry = (carry - cin) + (x - nv);
                    }
                    if constexpr (LAST) {
                        const unsigned long long any = __ballot(nv >= smin);
                        sflag[t - 3] = any ? 1 : 0;
                    }
                }
            }
            a3d = aid;
            a2 = a1;
            a1 = a;
            da_prev = da;
            face_prev = face;
            Fc_prev = Fc;
            Ff_prev = Ff;
        }
        if (g == 0 && G > 1) build_next();
    }
}

template <int ST, bool LAST>
__device__ __forceinline__ void sweep_stream(const Dev &D, const SweepParams &sp)
{
    using C = typename std::conditional<ST == VL_F64, double, float>::type;
    __shared__ __align__(16) uint32_t s_tab[4][2][MAXL + 48];
    __shared__ uint8_t s_flg[4][MAXL + 48];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int d = sp.d, L = sp.L, WL = sp.WL;
    const int ld = (d == 0) ? (lane & 3) : (d == 1) ? ((lane >> 2) & 3) : (lane >> 4);
    const int64_t nitems = min((int64_t)D.ctl->n_items[sp.sidx], D.item_cap);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    int64_t it = (int64_t)blockIdx.x * 4 + wv;
    if (it >= nitems) return;
    uint32_t *X = s_tab[wv][0], *Y = s_tab[wv][1];
    uint8_t *sflag = s_flg[wv];
    int place = 0;  // X's blocks for the old values of the line's first cells; Y has the others
    build_slots<ST>(D, it, nitems, L, WL, sp.wrap, place, lane, X);
    wave_sync_lds();
    const uint32_t zslot = (uint32_t)D.trash;
    constexpr int BS = Storage<ST>::BYTES;
    C q[8];
#pragma unroll
    for (int u = 0; u < 8; u++) {
        uint32_t sl = uniform_u32(X[u]);
        sl = (sl & NEWFLAG) ? zslot : sl;
        const char *blk = (const char *)D.pool + (uint64_t)sl * (BLK * BS) + (uint32_t)lane * BS;
        if constexpr (ST == VL_F64)
            q[u] = *(const double *)blk;
        else if constexpr (ST == VL_F32)
            q[u] = *(const float *)blk;
        else
            q[u] = bf16_to_f32(*(const uint16_t *)blk);
    }
    for (; it < nitems; it += nwaves) {
        const int64_t nit = it + nwaves;
        const double c = courant(D, d, 4 * D.items[it].key + ld, sp.dt);
        const unsigned long long npos = __ballot(c > 0.0), nneg = __ballot(c < 0.0);
        int32_t src = -1;
        if constexpr (ST != VL_F64)
            if (it < sp.lg_cap) src = sp.lg_src[it];
        const double start_sum = take_residual<ST>(sp, (int32_t)uniform_u32((uint32_t)src));
        double carry = start_sum * (1.0 / BLK);
        auto build = [&]() {
            build_slots<ST>(D, nit, nitems, L, WL, sp.wrap, WRAP - place, lane, Y);
            wave_sync_lds();
        };
        if (npos == ~0ull)
            march_stream<ST, 1, LAST>(D, X, Y, sflag, L, c, lane, sp.sparse_min, carry, q, build);
        else if (nneg == ~0ull)
            march_stream<ST, -1, LAST>(D, X, Y, sflag, L, c, lane, sp.sparse_min, carry, q, build);
        else
            march_stream<ST, 0, LAST>(D, X, Y, sflag, L, c, lane, sp.sparse_min, carry, q, build);
        if constexpr (LAST) {
            wave_sync_lds();
            store_flag_words(D, it, X, sflag, L, lane);
        }
        leave_residual<ST>(D, sp, it, lane, carry, start_sum);  // the line's final carry
        wave_sync_lds();
        uint32_t *tmp = X;
        X = Y;
        Y = tmp;
        place = WRAP - place;
    }
}

template <int ST, bool LAST, int V, int NM>
__global__ __launch_bounds__(256) void k_sweep(Dev D, SweepParams sp)
{
    if (failed(D)) return;  // waves are independent: no barrier to keep
    if constexpr (VARIANTS[V].style == 2)
        sweep_stream<ST, LAST>(D, sp);
    else
        sweep_body<ST, LAST, V, NM>(D, sp);
}

template <int ST, bool LAST, int V, int NM, int MINW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MINW))) void k_sweep_occ(Dev D, SweepParams sp)
{
    if (failed(D)) return;
    if constexpr (VARIANTS[V].style == 2)
        sweep_stream<ST, LAST>(D, sp);
    else
        sweep_body<ST, LAST, V, NM>(D, sp);
}

template <typename K>
static dim3 persistent_grid(K kernel)
{
    // exactly the workgroups that fit on the device at once, so every
    // wavefront's share of the static item assignment runs in one round
    static int ncu = 0;
    if (ncu == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            ncu = 256;
    }
    int per = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, 256, 0) != hipSuccess || per < 1) per = 1;
    // (each wavefront has blocks of its own in the pool: NSINK in all)
    return dim3((unsigned)std::min(per * ncu, NSINK / 4));
}

template <int ST, bool LAST, int V, int NM>
static void launch_words(const Dev &D, const SweepParams &sp, hipStream_t st)
{
    constexpr VariantInfo vi = VARIANTS[V];
    if constexpr (vi.minw > 0) {
        static const dim3 g = persistent_grid(k_sweep_occ<ST, LAST, V, NM, (vi.minw > 0 ? vi.minw : 1)>);
        hipLaunchKernelGGL((k_sweep_occ<ST, LAST, V, NM, (vi.minw > 0 ? vi.minw : 1)>), g, dim3(256), 0, st, D, sp);
    } else {
        static const dim3 g = persistent_grid(k_sweep<ST, LAST, V, NM>);
        hipLaunchKernelGGL((k_sweep<ST, LAST, V, NM>), g, dim3(256), 0, st, D, sp);
    }
}

// the kernel for the line's mask words (the streamed and unconditional
// variants hold the longest line's)
template <int ST, bool LAST, int V>
static void launch_variant(const Dev &D, const SweepParams &sp, hipStream_t st)
{
    if constexpr (VARIANTS[V].style == 0) {
        if (sp.L <= 64) return launch_words<ST, LAST, V, 1>(D, sp, st);
        if (sp.L <= 128) return launch_words<ST, LAST, V, 2>(D, sp, st);
    }
    launch_words<ST, LAST, V, MAXL / 64>(D, sp, st);
}

template <int ST, bool LAST>
static void launch_st(const Dev &D, const SweepParams &sp, int v, hipStream_t st)
{
    switch (v) {
    case 1: launch_variant<ST, LAST, 1>(D, sp, st); break;
    case 2: launch_variant<ST, LAST, 2>(D, sp, st); break;
    case 3: launch_variant<ST, LAST, 3>(D, sp, st); break;
    case 4: launch_variant<ST, LAST, 4>(D, sp, st); break;
    case 5: launch_variant<ST, LAST, 5>(D, sp, st); break;
    case 6: launch_variant<ST, LAST, 6>(D, sp, st); break;
    case 7: launch_variant<ST, LAST, 7>(D, sp, st); break;
    case 8: launch_variant<ST, LAST, 8>(D, sp, st); break;
    case 9: launch_variant<ST, LAST, 9>(D, sp, st); break;
    case 10: launch_variant<ST, LAST, 10>(D, sp, st); break;
    default: launch_variant<ST, LAST, 0>(D, sp, st); break;
    }
}

int sweep_variants() { return NVARIANTS; }

void launch_sweep(const Dev &D, int d, int sidx, const int lo[3], const int hi[3], double dt, bool last,
                  const LedgerIO &lg, bool wrap, hipStream_t st)
{
    SweepParams sp;
    sp.wrap = wrap ? D.n[d] : 0;
    sp.lg_old = lg.old.res;
    sp.lg_new = lg.nw.res;
    sp.lg_src = lg.src;
    sp.lg_cap = lg.src ? lg.cap : 0;
    sp.d = d;
    sp.sidx = sidx;
    sp.L = D.P[d];
    sp.WL = (sp.L + 31) / 32;
    sp.dt = dt;
    sp.sparse_min = D.sparse_min;
    const int v = (D.sweep_variant[sidx] >= 0 && D.sweep_variant[sidx] < NVARIANTS) ? D.sweep_variant[sidx] : 0;
    switch (D.storage) {
    case VL_F64: last ? launch_st<VL_F64, true>(D, sp, v, st) : launch_st<VL_F64, false>(D, sp, v, st); break;
    case VL_F32: last ? launch_st<VL_F32, true>(D, sp, v, st) : launch_st<VL_F32, false>(D, sp, v, st); break;
    default: last ? launch_st<VL_BF16, true>(D, sp, v, st) : launch_st<VL_BF16, false>(D, sp, v, st); break;
    }
}

// ---------------------------------------------------------------------------
// mass ledger of one shear: the terminal residuals of the local pencils'
// items, summed per pencil over its items (ascending block id) by one
// wavefront, then over the pencils in order by one workgroup; no atomics, so
// the total is the same in every run
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_ledger_pencils(Dev D, int e1, int e2, int lo1, int n1, int lo2,
                                                        int64_t npen, double *pen_sum)
{
    const int lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (p >= npen || failed(D)) return;
    const int t1 = lo1 + (int)(p % n1), t2 = lo2 + (int)(p / n1);
    const bool local = t1 >= H && t1 < H + D.n[e1] && t2 >= H && t2 < H + D.n[e2];
    double acc = 0.0;
    if (local && p < D.pen_cap) {
        const int64_t first = D.pen_first[p];
        const int64_t cnt = min((int64_t)D.pen_cnt[p], max((int64_t)0, D.item_cap - first));
        for (int64_t k = lane; k < cnt; k += 64) acc += D.resid[first + k];
    }
    acc = wave_sum_f64(acc);
    if (lane == 0) pen_sum[p] = acc;
}

__global__ __launch_bounds__(1024) void k_sum_fixed(const double *in, int64_t n, double *out)
{
    __shared__ double s[1024];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) acc += in[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

void launch_ledger_sum(const Dev &D, int d, const int lo[3], const int hi[3], double *out, hipStream_t st)
{
    const int e1 = (d == 0) ? 1 : 0, e2 = (d == 2) ? 1 : 2;
    const int n1 = hi[e1] - lo[e1], n2 = hi[e2] - lo[e2];
    const int64_t npen = (int64_t)n1 * n2;
    if (npen <= 0 || D.storage == VL_F64) {
        hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, st, D.cell_red, (int64_t)0, out);
        return;
    }
    // per-pencil sums in the scratch of per-cell sums (npen <= padded cells)
    hipLaunchKernelGGL(k_ledger_pencils, dim3((unsigned)((npen + 3) / 4)), dim3(256), 0, st, D, e1, e2, lo[e1],
                       n1, lo[e2], npen, D.pen_sum);
    hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, st, D.pen_sum, npen, out);
}

}  // namespace vl
