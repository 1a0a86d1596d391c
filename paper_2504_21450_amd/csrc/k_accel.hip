// Acceleration step: the Lorentz-force term of the Vlasov equation over one
// time step (Section 2, eq. 1; the velocity-space half of the split step),
// as the three one-coordinate remaps of SLICE-3D (Zerroukat & Allen 2012).
//
// In fields E, B that are constant over the step every velocity moves along
// the exact characteristic of dv/dt = (q/m)(E + v x B): the affine map
// v' = A v + c with A the rotation by -(q/m)|B| dt about B/|B| (Rodrigues)
// and c = (I - A) vE + (q/m)(E.b) dt b (vE = E x B / |B|^2; with B = 0,
// v' = v + (q/m) E dt).  SLICE-3D writes the map as three maps that each set
// one coordinate to its final value as an affine function of the current
// coordinates (rows of the homogeneous form times the inverses of the maps
// before), so the three compose to the map exactly.  Each is a remap of every
// velocity column along its axis: a column moves by u -> alpha u + sigma in
// cell units, and cell i receives the mass of its pre-image under the CW84
// parabolas of the column (the slopes, faces and limiter of the spatial
// remap), cells outside the velocity mesh reading as zero.
//
// k_accel_factors: per local cell, the three maps (12 doubles) and a flag if a
//   map cannot be split (its own coefficient not positive).
// Per remap, along axis d, two kernels:
// k_accel_plan, one workgroup per local cell: a block column (fixed block
//   coordinates across d) spans from its lowest to its highest block, widened
//   to where its image can reach (the map of the column's extent with the
//   extreme shifts of its 16 velocity columns, one cell of margin); blocks of
//   that span missing from the cell are created: slots from the free ring,
//   entries merged into the sorted list (in place from the end, or into a
//   larger place when the list outgrows it).  Every block column becomes a
//   work item with a row of the list places of its blocks.
// k_accel_remap, one wavefront per block column, persistent: it stages the
//   column in LDS in the storage type (16 velocity columns x its span, missing
//   blocks as zero), then takes the column's faces four cells of sixteen
//   columns at a time: the departure point of a cell's lower face, the limited
//   parabola of the source cell it lies in and that parabola's head, once per
//   face; a cell's new average takes its upper face from the next lane of its
//   quad (lanes: quad = the 4 cells of a velocity column in the block), so each
//   head is computed once.  Blocks are read and written whole.
//   The last remap leaves per list entry the flags the pruning reads: bit 0 a
//   value >= the content threshold, bit 1 a nonzero value, bit 2 created by
//   this step.
// Blocks created but left all zero are dropped by the pruning (as the new
// block set is the old one plus every block holding a nonzero value).
// Before, one workgroup took a cell through all three remaps, a block column
// at a time with three barriers each: hot cells of a mixture (4,400 blocks
// beside 80) ran long after the rest, and every cell's columns were a serial
// chain.  Acceleration step with moments, before -> now: 24x24x12 BF16
// mixture 19.1 -> 6.2 ms, 11x9x7 sparse FP64 1.50 -> 0.66 ms.
#include <algorithm>

#include "vl_internal.h"
#include "vl_storage.h"

namespace vl {

struct AccelParams {
    const double *fields;  // per local cell Ex, Ey, Ez, Bx, By, Bz
    double *maps;          // per local cell 3 x 4 map rows (ACC_MAP doubles)
    int *bad;              // set if some cell's map cannot be split
    double qm, dt;
    int order[3];
    int cur;               // local list region in use
    int ncols;             // block columns of the widest cross-section
    int mx;                // blocks of the longest axis
    int64_t q0;            // first local cell of this launch
    uint32_t mg[2];        // ceil(2^32 / nblk[0 / 1]): exact division of block ids (below 2^17, by at most 2^10)
};

constexpr int ACC_MAP = ACC_MAP_DOUBLES;

// ---------------------------------------------------------------------------
// per-cell maps
// ---------------------------------------------------------------------------
// identity with row d replaced by `row`, inverted (4x4 homogeneous)
__device__ inline void inv_row_step(const double *row, int d, double (&Mi)[4][4])
{
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) Mi[i][j] = (i == j) ? 1.0 : 0.0;
    for (int j = 0; j < 4; j++) Mi[d][j] = (j == d) ? 1.0 / row[d] : -row[j] / row[d];
}

__device__ inline void row_mul(const double *row, const double (&M)[4][4], double *out)
{
    for (int j = 0; j < 4; j++) {
        double s = 0.0;
        for (int i = 0; i < 4; i++) s += row[i] * M[i][j];
        out[j] = s;
    }
}

__global__ __launch_bounds__(256) void k_accel_factors(Dev D, AccelParams ap)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= D.nlocal) return;
    const double *EB = ap.fields + 6 * q;
    const double E[3] = {EB[0], EB[1], EB[2]}, B[3] = {EB[3], EB[4], EB[5]};
    double T[3][4];
    const double Bm = sqrt(B[0] * B[0] + B[1] * B[1] + B[2] * B[2]);
    if (Bm == 0.0) {
        for (int i = 0; i < 3; i++) {
            for (int j = 0; j < 3; j++) T[i][j] = (i == j) ? 1.0 : 0.0;
            T[i][3] = ap.qm * E[i] * ap.dt;
        }
    } else {
        const double b[3] = {B[0] / Bm, B[1] / Bm, B[2] / Bm};
        const double th = -ap.qm * Bm * ap.dt;
        double si, co;
        sincos(th, &si, &co);
        // [b]x: the matrix of v -> b x v
        const double K[3][3] = {{0.0, -b[2], b[1]}, {b[2], 0.0, -b[0]}, {-b[1], b[0], 0.0}};
        for (int i = 0; i < 3; i++)
            for (int j = 0; j < 3; j++) T[i][j] = ((i == j) ? co : 0.0) + si * K[i][j] + (1.0 - co) * b[i] * b[j];
        const double B2 = Bm * Bm;
        const double vE[3] = {(E[1] * B[2] - E[2] * B[1]) / B2, (E[2] * B[0] - E[0] * B[2]) / B2,
                              (E[0] * B[1] - E[1] * B[0]) / B2};
        const double Epar = E[0] * b[0] + E[1] * b[1] + E[2] * b[2];
        for (int i = 0; i < 3; i++) {
            const double Av = T[i][0] * vE[0] + T[i][1] * vE[1] + T[i][2] * vE[2];
            T[i][3] = vE[i] - Av + ap.qm * Epar * ap.dt * b[i];
        }
    }
    // the three one-coordinate maps in the slice order
    const int o0 = ap.order[0], o1 = ap.order[1], o2 = ap.order[2];
    double r0[4], r1[4], r2[4], t[4];
    double I0[4][4], I1[4][4];
    for (int j = 0; j < 4; j++) r0[j] = T[o0][j];
    bool ok = r0[o0] > 0.0;
    inv_row_step(r0, o0, I0);
    row_mul(T[o1], I0, r1);
    ok = ok && r1[o1] > 0.0;
    inv_row_step(r1, o1, I1);
    row_mul(T[o2], I0, t);
    row_mul(t, I1, r2);
    ok = ok && r2[o2] > 0.0;
    double *m = ap.maps + ACC_MAP * q;
    for (int j = 0; j < 4; j++) {
        m[j] = r0[j];
        m[4 + j] = r1[j];
        m[8 + j] = r2[j];
    }
    if (!ok) *ap.bad = 1;
}

// ---------------------------------------------------------------------------
// column remap
// ---------------------------------------------------------------------------
// twice the limited slope of a cell (CW84 eq. 1.7-1.8) from its one-sided
// differences dl, dr (given as x4, scaled exactly) and their sum c: c limited
// to four times either difference, zero at an extremum
__device__ __forceinline__ double col_slope2(double dl4, double dr4, double c)
{
    const double up = fmax(0.0, fmin(fmin(dl4, dr4), c));  // c > 0
    const double dn = fmin(0.0, fmax(fmax(dl4, dr4), c));  // c < 0
    return up + dn;                                        // (one of them is zero)
}

// CW84 eq. 1.10 on the face offsets: x limited to twice the other side's
// offset y, zero unless they share a sign
__device__ __forceinline__ double col_offset(double x, double y)
{
    return copysign(fmax(0.0, fmin(fabs(x), copysign(2.0, x) * y)), x);
}

// Mass of a source cell's limited parabola over [0, x] of the cell (0 <= x <=
// 1, cell units), from the averages of the five cells around it.  The face
// offsets dL = a - a_L, dR = a_R - a (CW84 eq. 1.6 faces) are formed from the
// differences, limited, and put into eq. 1.5's profile, whose integral is
//   x (a - dL + x (2 dL - dR - x (dL - dR))).
// The limiter's minima and maxima pass over a NaN, so the neighbours'
// difference enters once more, times zero: a parabola next to a NaN is none.
__device__ __forceinline__ double col_head(double am2, double am, double a0, double ap, double ap2, double x)
{
    constexpr double TWELFTH = 1.0 / 12.0;
    const double g0 = am - am2, g1 = a0 - am, g2 = ap - a0, g3 = ap2 - ap;
    const double h0 = 4.0 * g0, h1 = 4.0 * g1, h2 = 4.0 * g2, h3 = 4.0 * g3;
    const double dm = col_slope2(h0, h1, a0 - am2), d0 = col_slope2(h1, h2, ap - am), dp = col_slope2(h2, h3, ap2 - a0);
    const double dL = fma(0.5, g1, (d0 - dm) * TWELFTH), dR = fma(0.5, g2, (d0 - dp) * TWELFTH);
    const double l = col_offset(dL, dR), r = col_offset(dR, dL);
    return x * fma(x, fma(-x, l - r, fma(2.0, l, -r)), fma(0.0, ap - am, a0) - l);
}

// shift sigma (cell units) of the velocity column at transverse velocity
// indices (i1, i2) under map row `row` along d
__device__ inline double col_sigma(const Dev &D, const double *row, int d, int e1, int e2, int i1, int i2)
{
#pragma clang fp contract(off)
    const double w1 = D.vmin[e1] + ((double)i1 + 0.5) * D.dv[e1];
    const double w2 = D.vmin[e2] + ((double)i2 + 0.5) * D.dv[e2];
    const double s = row[e1] * w1 + row[e2] * w2 + row[3];
    return ((row[d] - 1.0) * D.vmin[d] + s) / D.dv[d];
}

__device__ inline int32_t compose_id(const Dev &D, int d, int e1, int e2, int bd, int b1, int b2)
{
    int c[3];
    c[d] = bd;
    c[e1] = b1;
    c[e2] = b2;
    return c[0] + D.nblk[0] * (c[1] + D.nblk[1] * c[2]);
}

__device__ inline bool has_bit(const uint32_t *bm, int32_t id) { return (bm[id >> 5] >> (id & 31)) & 1u; }

__device__ inline int rank_of(const uint32_t *bm, const int *rk, int32_t id)
{
    return rk[id >> 5] + __popc(bm[id >> 5] & ((1u << (id & 31)) - 1u));
}

// inclusive sums of v over the workgroup's threads before and with this one;
// the total of all in `total` (s_w: one entry per wavefront)
__device__ __forceinline__ int block_incl(int v, int *s_w, int &total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    if (lane == 63) s_w[wv] = v;
    __syncthreads();
    total = 0;
    for (int w = 0; w < 4; w++) {
        const int t = s_w[w];
        v += w < wv ? t : 0;
        total += t;
    }
    return v;
}

// a row entry: the block's place in the cell's list, created in this step
// (zero in the cell's state before it) and in this remap (reads as zero)
constexpr uint32_t ROW_PLACE = 0x3ffff, ROW_STEP = 0x40000000u, ROW_NEW = 0x80000000u;
static_assert(NB_MAX <= 0x40000, "list place in a row entry");

// a work item's block column: lowest and highest block and the column's number
__device__ inline int32_t pack_column(int col, int lo, int hi) { return col | (lo << 12) | (hi << 18); }
static_assert(ACC_MAX_NBLK <= 64, "six bits a block coordinate");

// Bound by latency: a dozen barriers and four dependent reads of the list.
// Spans come from one LDS minimum, maximum and count per list entry, not from
// a test of every block of the mesh.
__global__ __launch_bounds__(256) void k_accel_plan(Dev D, AccelParams ap, int k)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_w[4][4];
    __shared__ int s_cnt[2];
    __shared__ long long s_at[2];
    __shared__ unsigned long long s_base[3];
    __shared__ int s_fail;
    const int tid = threadIdx.x;
    const int W = D.W;
    uint32_t *s_bm = (uint32_t *)smem;     // block set after this remap's creations
    uint32_t *s_old = s_bm + W;            // and before
    int *s_rank = (int *)(s_old + W);      // W + 1
    int *s_lo = s_rank + (W + 1);          // per block column: lowest block, then lo | hi << 16, or -1
    int *s_hi = s_lo + ap.ncols;           // highest block, then blocks to create
    int *s_len = s_hi + ap.ncols;          // blocks held, then row entries before it

    const int64_t q = ap.q0 + blockIdx.x;
    const int x = (int)(q % D.n[0]), y = (int)((q / D.n[0]) % D.n[1]), z = (int)(q / ((int64_t)D.n[0] * D.n[1]));
    const int64_t c = cell_index(D, x + H, y + H, z + H);
    const int d = ap.order[k];
    const int e1 = (d == 0) ? 1 : 0, e2 = (d == 2) ? 1 : 2;
    const int nbd = D.nblk[d], nb1 = D.nblk[e1], nb2 = D.nblk[e2];
    const int N = 4 * nbd;
    const int ncol = nb1 * nb2;
    double row[4];
    for (int j = 0; j < 4; j++) row[j] = ap.maps[ACC_MAP * q + 4 * k + j];
    const double alpha = row[d];
    if (tid == 0) {
        s_fail = failed(D) ? 1 : 0;
        s_at[0] = D.lstart[c];
        s_cnt[0] = D.lcount[c];
        s_cnt[1] = D.lcapa[c];
    }
    for (int w = tid; w < W; w += 256) s_bm[w] = 0u;
    for (int col = tid; col < ncol; col += 256) {
        s_lo[col] = nbd;
        s_hi[col] = -1;
        s_len[col] = 0;
    }
    __syncthreads();
    if (s_fail) return;
    const int cnt = s_cnt[0], cap = s_cnt[1];
    const int64_t cs = s_at[0];
    // block coordinates along d and across
    auto place = [&](int32_t id, int &bd) -> int {
        const int r = D.nblk[0] > 1 ? (int)__umulhi((uint32_t)id, ap.mg[0]) : id;
        const int b2 = D.nblk[1] > 1 ? (int)__umulhi((uint32_t)r, ap.mg[1]) : r;
        const int b0 = id - r * D.nblk[0], b1 = r - b2 * D.nblk[1];
        bd = d == 0 ? b0 : d == 1 ? b1 : b2;
        return (e1 == 0 ? b0 : b1) + nb1 * (e2 == 1 ? b1 : b2);
    };
    // 1. block set, and per column its extent and count
    constexpr int MU = 4;  // entries a thread takes at a time, their loads together
    for (int e0 = tid; e0 < cnt; e0 += 256 * MU) {
        int32_t id[MU];
#pragma unroll
        for (int u = 0; u < MU; u++) id[u] = e0 + 256 * u < cnt ? D.lid[cs + e0 + 256 * u] : -1;
#pragma unroll
        for (int u = 0; u < MU; u++) {
            if (id[u] < 0) continue;
            int bd;
            const int col = place(id[u], bd);
            atomicOr(&s_bm[id[u] >> 5], 1u << (id[u] & 31));
            atomicMin(&s_lo[col], bd);
            atomicMax(&s_hi[col], bd);
            atomicAdd(&s_len[col], 1);
        }
    }
    __syncthreads();
    for (int w = tid; w < W; w += 256) s_old[w] = s_bm[w];
    // 2. spans; a thread takes a run of consecutive columns
    const int per = (ncol + 255) / 256;
    const int c0 = min(tid * per, ncol), c1 = min(c0 + per, ncol);
    int my_new = 0, my_row = 0, my_items = 0;
    for (int col = c0; col < c1; col++) {
        const int bmin = s_lo[col], bmax = s_hi[col], have = s_len[col];
        if (have == 0) {
            s_lo[col] = -1;
            s_hi[col] = 0;
            continue;
        }
        const int b1 = col % nb1, b2 = col / nb1;
        // extreme shifts: sigma is affine in the velocity column, so at
        // the corners of the block column's 4 x 4
        double smin = 1e300, smax = -1e300;
        for (int u = 0; u < 4; u++) {
            const double s = col_sigma(D, row, d, e1, e2, 4 * b1 + 3 * (u & 1), 4 * b2 + 3 * (u >> 1));
            smin = fmin(smin, s);
            smax = fmax(smax, s);
        }
        // cells that can receive mass from [4 bmin, 4 bmax + 4): those
        // with alpha u0 + sigma - 1 < i < alpha u1 + sigma (a cell of margin)
        const double ilo = floor(alpha * (4.0 * bmin) + smin) - 1.0;
        const double ihi = ceil(alpha * (4.0 * bmax + 4.0) + smax);
        int lo = bmin, hi = bmax;
        if (ihi >= 0.0 && ilo <= (double)(N - 1)) {
            const int i0 = (int)fmax(ilo, 0.0), i1 = (int)fmin(ihi, (double)(N - 1));
            lo = min(lo, i0 >> 2);
            hi = max(hi, i1 >> 2);
        }
        const int len = hi - lo + 1;
        s_lo[col] = lo | (hi << 16);
        s_hi[col] = len - have;
        s_len[col] = len;
        my_new += len - have;
        my_row += len;
        my_items++;
    }
    int T, R, I;
    block_incl(my_new, s_w[0], T);
    int run_row = block_incl(my_row, s_w[1], R) - my_row;
    int run_item = block_incl(my_items, s_w[2], I) - my_items;
    // 3. places: items and rows, slots for the created blocks, a larger list
    //    place if needed
    if (tid == 0) {
        unsigned long long err = 0;
        s_at[1] = cs;
        s_base[0] = I > 0 ? atomicAdd(&D.ctl->acc_items[k], (unsigned long long)I) : 0ull;
        s_base[1] = R > 0 ? atomicAdd(&D.ctl->acc_rows[k], (unsigned long long)R) : 0ull;
        s_base[2] = 0ull;
        if ((int64_t)(s_base[0] + I) > D.item_cap) err |= E_ITEMS;  // (not reached: launch_accel sizes its launches)
        if ((int64_t)(s_base[1] + R) > D.row_cap) err |= E_ROWS;    // (not reached: rows hold blocks with slots)
        if (T > 0) {
            const unsigned long long nb = atomicAdd(&D.ctl->ring_head, (unsigned long long)T);
            if (nb + T > D.ctl->ring_limit) err |= E_RING;
            s_base[2] = nb;
            if (cnt + T > cap) {
                const int ncap = (cnt + T) + (cnt + T) / 2 + 32;
                const unsigned long long nb0 = atomicAdd(&D.ctl->list_top[ap.cur], (unsigned long long)ncap);
                if ((int64_t)(nb0 + ncap) > D.reg_cap[ap.cur]) err |= E_LOCAL_LIST;
                s_at[1] = D.reg_off[ap.cur] + (int64_t)nb0;
                s_cnt[1] = ncap;
            }
        }
        // (a full ring is the error to report where rows are short as well)
        if (err & E_RING) err &= ~(unsigned long long)E_ROWS;
        if (err) atomicOr(&D.ctl->err, err);
        s_fail = err ? 1 : 0;
    }
    __syncthreads();
    if (s_fail) return;  // the partition is reported as failed; nothing is read again
    const int64_t ns = s_at[1];
    const int64_t rb = (int64_t)s_base[1];
    for (int col = c0; col < c1; col++) {
        const int sp = s_lo[col], nw = s_hi[col], len = s_len[col];
        s_len[col] = run_row;
        if (sp >= 0) {
            Item it;
            it.id = pack_column(col, sp & 0xffff, sp >> 16);
            it.key = (int32_t)q;
            it.rowoff = rb + run_row;
            D.items[(int64_t)s_base[0] + run_item] = it;
            run_item++;
            run_row += len;
            if (nw > 0) {  // the created blocks join the set
                const int b1 = col % nb1, b2 = col / nb1;
                for (int bd = sp & 0xffff; bd <= (sp >> 16); bd++) {
                    const int32_t id = compose_id(D, d, e1, e2, bd, b1, b2);
                    if (!has_bit(s_old, id)) atomicOr(&s_bm[id >> 5], 1u << (id & 31));
                }
            }
        }
    }
    __syncthreads();
    // row entry of the block of list place pos
    auto put_row = [&](int32_t id, int pos, uint32_t flags) {
        int bd;
        const int col = place(id, bd);
        D.rows[rb + s_len[col] + (bd - (s_lo[col] & 0xffff))] = (int32_t)((uint32_t)pos | flags);
    };
    if (T == 0) {
        for (int e0 = tid; e0 < cnt; e0 += 256 * MU) {
            int32_t id[MU], fl[MU];
#pragma unroll
            for (int u = 0; u < MU; u++) {
                const int e = e0 + 256 * u;
                id[u] = e < cnt ? D.lid[cs + e] : -1;
                fl[u] = e < cnt && k > 0 ? D.litem[cs + e] : 0;
            }
#pragma unroll
            for (int u = 0; u < MU; u++) {
                if (id[u] < 0) continue;
                const int e = e0 + 256 * u;
                if (k == 0) D.litem[cs + e] = 0;  // bit 2: created in this step
                put_row(id[u], e, (fl[u] & 4) ? ROW_STEP : 0u);
            }
        }
        return;
    }
    // 4. ranks; the list is merged in id order (old entries move up to their
    //    new rank, from the end so that no entry is overwritten before it is
    //    read)
    {
        const int perw = (W + 255) / 256;
        const int w0 = min(tid * perw, W), w1 = min(w0 + perw, W);
        int sum = 0, total;
        for (int w = w0; w < w1; w++) sum += __popc(s_bm[w]);
        int run = block_incl(sum, s_w[3], total) - sum;
        for (int w = w0; w < w1; w++) {
            s_rank[w] = run;
            run += __popc(s_bm[w]);
        }
    }
    __syncthreads();
    for (int e_hi = cnt; e_hi > 0; e_hi -= 256 * MU) {
        int32_t id[MU], slot[MU], fl[MU];
#pragma unroll
        for (int u = 0; u < MU; u++) {
            const int e = e_hi - 1 - tid - 256 * u;
            id[u] = e >= 0 ? D.lid[cs + e] : -1;
            slot[u] = e >= 0 ? D.lslot[cs + e] : 0;
            fl[u] = e >= 0 && k > 0 ? D.litem[cs + e] : 0;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MU; u++) {
            if (id[u] < 0) continue;
            const int pos = rank_of(s_bm, s_rank, id[u]);
            D.lid[ns + pos] = id[u];
            D.lslot[ns + pos] = slot[u];
            D.litem[ns + pos] = fl[u];
            put_row(id[u], pos, (fl[u] & 4) ? ROW_STEP : 0u);
        }
        __syncthreads();
    }
    // the created blocks, a thread the words w0 .. w1 - 1 of the set: the
    // slots in id order
    {
        const int perw = (W + 255) / 256;
        const int w0 = min(tid * perw, W), w1 = min(w0 + perw, W);
        int sum = 0, total;
        for (int w = w0; w < w1; w++) sum += __popc(s_bm[w] & ~s_old[w]);
        unsigned long long kk = s_base[2] + (unsigned long long)(block_incl(sum, s_w[0], total) - sum);
        for (int w = w0; w < w1; w++) {
            const uint32_t bm = s_bm[w];
            uint32_t cr = bm & ~s_old[w];
            while (cr) {
                const int bit = __ffs(cr) - 1;
                cr &= cr - 1;
                const int pos = s_rank[w] + __popc(bm & ((1u << bit) - 1u));
                D.lid[ns + pos] = 32 * w + bit;
                D.lslot[ns + pos] = D.ring[(int64_t)(kk % (unsigned long long)D.lcap)];
                D.litem[ns + pos] = 4;
                kk++;
                put_row(32 * w + bit, pos, ROW_NEW | ROW_STEP);
            }
        }
    }
    if (tid == 0) {
        D.lstart[c] = ns;
        D.lcount[c] = cnt + T;
        D.lcapa[c] = s_cnt[1];
        D.lsorted[c] = cnt + T;
    }
}

__device__ inline void acc_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the value of the next lane of the quad, the quad's first lane giving `wrap`
// to its last
__device__ __forceinline__ int quad_next(int v, int wrap, bool first)
{
    return __builtin_amdgcn_mov_dpp(first ? wrap : v, 0x39, 0xf, 0xf, true);  // quad_perm 1 2 3 0
}
__device__ __forceinline__ double quad_next(double v, double wrap, bool first)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, v), b = __builtin_bit_cast(uint64_t, wrap);
    const uint32_t lo = (uint32_t)quad_next((int)(uint32_t)a, (int)(uint32_t)b, first);
    const uint32_t hi = (uint32_t)quad_next((int)(uint32_t)(a >> 32), (int)(uint32_t)(b >> 32), first);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// cells from one velocity column to the next in a column's LDS: the span, four
// zero cells before and after, an odd multiple of 4
__host__ __device__ inline int acc_stride(int mx) { return 4 * ((mx + 2) | 1); }

// In BF16 bound by vector instructions: a remap of the 6.0 million blocks,
// created ones included, of a 24x24x12 mixture takes 1.5 ms at 118 instructions
// a block, 75 % of the issue slots (its bytes, read and written once, take 0.35
// ms).  It was 171 instructions, and a step 8.8 instead of 7.5 ms, before a
// face's five cells lay at one address with offsets and the parabola was put in
// face offsets (fewer roundings, too: the error against 64 bits on 11x9x7 FP64
// cells went from 5.0e-15 to 4.6e-15).  In FP64 it is bound by latency: 47 % of
// the issue slots and 2.3 TB/s on 11x9x7 sparse cells (0.12 ms for 0.29 million
// blocks), as a column of a mesh 25 blocks long takes 13.8 KB of LDS and a
// compute unit so holds 11 wavefronts.  A workgroup is one wavefront, so the
// columns in LDS, 16 acc_stride values of the storage type each, pack a compute
// unit's 160 KiB without a remainder.
template <int ST>
__global__ __launch_bounds__(64) void k_accel_remap(Dev D, AccelParams ap, int k)
{
    using St = Storage<ST>;
    using T = typename St::T;
    extern __shared__ __align__(16) unsigned char smem[];
    if (failed(D)) return;
    const int lane = threadIdx.x;
    T *s_a = (T *)smem;
    const int d = ap.order[k];
    const int e1 = (d == 0) ? 1 : 0, e2 = (d == 2) ? 1 : 2;
    const int nb1 = D.nblk[e1];
    const bool last = k == 2;
    // lane = 4 x velocity column + cell along d; its value in a block
    const int ld = lane & 3, l1 = (lane >> 2) & 3, l2 = lane >> 4;
    const bool first = ld == 0;
    const int mem = (ld << (2 * d)) + (l1 << (2 * e1)) + (l2 << (2 * e2));
    const uint32_t off = (uint32_t)mem * St::BYTES;
    // cell j of velocity column c lies at c S + 4 + j: a face's five cells are
    // one address and offsets; S is an odd multiple of 4, so the quads of a
    // wavefront fall on different banks
    const int S = acc_stride(ap.mx);
    T *col_a = s_a + (lane >> 2) * S + 4;
    const int64_t nitems = min((int64_t)D.ctl->acc_items[k], D.item_cap);
    col_a[ld - 4] = (T)0;  // the block before every column
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const Item item = D.items[it];
        const int32_t pk = __builtin_amdgcn_readfirstlane(item.id);
        const uint32_t q = (uint32_t)__builtin_amdgcn_readfirstlane(item.key);
        const int col = pk & 0xfff, lo = (pk >> 12) & 63, hi = (pk >> 18) & 63;
        const int n = hi - lo + 1;
        const uint32_t yz = q / (uint32_t)D.n[0], z = yz / (uint32_t)D.n[1];
        const int64_t ls = D.lstart[cell_index(D, (int)(q - yz * D.n[0]) + H, (int)(yz - z * D.n[1]) + H, (int)z + H)];
        // lane u: list place and slot of the column's block u
        const uint32_t ent = lane < n ? (uint32_t)D.rows[item.rowoff + lane] : 0u;
        const int pos = (int)(ent & ROW_PLACE);
        const uint32_t slot = lane < n ? (uint32_t)D.lslot[ls + pos] : 0u;
        const uint32_t code = slot | ((ent & ROW_NEW) ? NEWFLAG : 0u);
        double row[4];
#pragma unroll
        for (int j = 0; j < 4; j++) row[j] = ap.maps[ACC_MAP * (int64_t)q + 4 * k + j];
        const double inv_alpha = 1.0 / row[d];
        const double sigma = col_sigma(D, row, d, e1, e2, 4 * (col % nb1) + l1, 4 * (col / nb1) + l2);
        // the column's values, eight blocks' loads in flight (created blocks
        // read as zero), and the block after it
        for (int u0 = 0; u0 < n; u0 += 8) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane((int)code, min(u0 + u, n - 1));
                v[u] = block_load_raw<ST>(block_rsrc_if<ST>(D.pool, sl, (int32_t)sl >= 0), off);
            }
#pragma unroll
            for (int u = 0; u < 8; u++)
                if (u0 + u < n) col_a[4 * (u0 + u) + ld] = v[u];
        }
        col_a[4 * n + ld] = (T)0;
        acc_wave_sync();
        const int base = 4 * lo, ncell = 4 * n;
        // average of the column's cell j (relative to base, -4 <= j < ncell + 4)
        auto a = [&](int j) -> double { return St::widen(col_a[j]); };
        int jp = 0, fl = 0;
        double hp = 0.0, ap0 = 0.0;  // the lower faces of the block before: source cell, head, its average
        for (int b = 0; b <= n; b++) {
            // lower face of cell base + 4 b + ld: its departure point lies in
            // source cell j, a fraction xf above the cell's lower edge
            double xd = ((double)(base + 4 * b + ld) - sigma) * inv_alpha;
            xd = fmin(fmax(xd, (double)(base - 1)), (double)(base + ncell + 1));
            const double f = floor(xd);
            const int j = (int)f - base;
            const double xf = xd - f;
            const double a0 = a(j);
            const double hd = col_head(a(j - 2), a(j - 1), a0, a(j + 1), a(j + 2), xf);
            // cells outside the span hold zero: flat zero parabolas
            const double h = (unsigned)j < (unsigned)ncell && xf > 0.0 ? hd : 0.0;
            if (b > 0) {
                // new averages of block b - 1: the tail of the first source
                // cell, the cells covered whole, the head of the last
                const int j1 = quad_next(jp, j, first);
                const double h1 = quad_next(hp, h, first);
                double v = jp == j1 ? h1 - hp : ap0 - hp;
                if (jp != j1) {
                    for (int m = jp + 1; m < j1; m++) v += a(m);
                    v += h1;
                }
                const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane((int)slot, b - 1);
                if constexpr (ST == VL_F64)
                    block_store(block_rsrc<ST>(D.pool, sl), off, v);
                else if constexpr (ST == VL_F32)
                    block_store(block_rsrc<ST>(D.pool, sl), off, (float)v);
                else
                    block_store(block_rsrc<ST>(D.pool, sl), off, St::encode(v));
                if (last) {
                    const double sv = St::round(v);
                    const unsigned long long bc = __ballot(sv >= D.sparse_min), bz = __ballot(sv != 0.0);
                    if (lane == b - 1) fl = (bc ? 1 : 0) | (bz ? 2 : 0);
                }
            }
            jp = j;
            hp = h;
            ap0 = a0;
        }
        if (last && lane < n) D.litem[ls + pos] = fl | ((ent & ROW_STEP) ? 4 : 0);
        acc_wave_sync();
    }
}

// The size by which a velocity mesh is accepted (see vl_accelerate), or 0 if an
// axis is beyond ACC_MAX_NBLK blocks: a cell's block sets, with a block column's
// averages and parabolas beside them.  Neither kernel holds both, so a mesh
// within it fits them: the planner 12 bytes per 32 blocks and 12 per column
// (77 KB at most), the remap 34 KB.
size_t accel_lds_bytes(const Dev &D, int *ncols, int *hc)
{
    int nc = 0, mx = 0;
    for (int d = 0; d < 3; d++) {
        const int e1 = (d == 0) ? 1 : 0, e2 = (d == 2) ? 1 : 2;
        nc = std::max(nc, D.nblk[e1] * D.nblk[e2]);
        mx = std::max(mx, D.nblk[d]);
    }
    if (mx > ACC_MAX_NBLK) return 0;
    *ncols = nc;
    *hc = 4 * mx;
    size_t b = sizeof(uint32_t) * (size_t)D.W * 3 + sizeof(int) * (size_t)(D.W + 1) + sizeof(int) * (size_t)nc * 2;
    b = (b + 15) & ~(size_t)15;
    return b + sizeof(double) * 3 * 16 * (size_t)(*hc + 1);
}

static AccelParams accel_params(const Dev &D, const double *fields, double *maps, int *bad, double qm, double dt,
                                const int order[3], int cur)
{
    AccelParams ap;
    ap.fields = fields;
    ap.maps = maps;
    ap.bad = bad;
    ap.qm = qm;
    ap.dt = dt;
    for (int k = 0; k < 3; k++) ap.order[k] = order[k];
    ap.cur = cur;
    ap.ncols = 0;
    ap.mx = 0;
    ap.q0 = 0;
    for (int j = 0; j < 2; j++)
        ap.mg[j] = (uint32_t)((((uint64_t)1 << 32) + D.nblk[j] - 1) / D.nblk[j]);  // (1 block: not used)
    return ap;
}

void launch_accel_maps(const Dev &D, const double *fields, double *maps, int *bad, double qm, double dt,
                       const int order[3], hipStream_t st)
{
    const AccelParams ap = accel_params(D, fields, maps, bad, qm, dt, order, 0);
    hipLaunchKernelGGL(k_accel_factors, dim3((unsigned)((D.nlocal + 255) / 256)), dim3(256), 0, st, D, ap);
}

template <int ST>
static void launch_remap(const Dev &D, const AccelParams &ap, int k, hipStream_t st)
{
    // one round of workgroups: as many wavefronts as a compute unit's LDS holds
    // columns for, and its registers wavefronts
    static const int ncu = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            n = 256;
        return n;
    }();
    const size_t lds = (size_t)16 * acc_stride(ap.mx) * Storage<ST>::BYTES;
    const int per = (int)std::max<size_t>(1, std::min<size_t>(32, (160 * 1024) / lds));
    hipLaunchKernelGGL(k_accel_remap<ST>, dim3((unsigned)(ncu * per)), dim3(64), lds, st, D, ap, k);
}

int launch_accel(const Dev &D, double *maps, const int order[3], int cur, hipStream_t st)
{
    AccelParams ap = accel_params(D, nullptr, maps, nullptr, 0.0, 0.0, order, cur);
    int hc = 0;
    if (accel_lds_bytes(D, &ap.ncols, &hc) == 0) return -1;
    ap.mx = hc / 4;
    const size_t lds = sizeof(uint32_t) * (size_t)D.W * 2 + sizeof(int) * ((size_t)D.W + 1 + 3 * (size_t)ap.ncols);
    // A remap has at most one item per block, which the item array holds in a
    // partition of up to 2^24 blocks; a larger one takes its cells in launches
    // whose columns are sure to fit.
    const int64_t tot = D.lcap + D.gcap;
    const int64_t step = D.item_cap >= tot ? D.nlocal : std::max<int64_t>(1, D.item_cap / ap.ncols);
    for (ap.q0 = 0; ap.q0 < D.nlocal; ap.q0 += step) {
        const int64_t ncell = std::min(step, D.nlocal - ap.q0);
        if (ap.q0 > 0) launch_book(D, BOOK_COLUMNS, st);
        for (int k = 0; k < 3; k++) {
            hipLaunchKernelGGL(k_accel_plan, dim3((unsigned)ncell), dim3(256), lds, st, D, ap, k);
            switch (D.storage) {
            case VL_F64: launch_remap<VL_F64>(D, ap, k, st); break;
            case VL_F32: launch_remap<VL_F32>(D, ap, k, st); break;
            default: launch_remap<VL_BF16>(D, ap, k, st); break;
            }
        }
    }
    return 0;
}

}  // namespace vl
