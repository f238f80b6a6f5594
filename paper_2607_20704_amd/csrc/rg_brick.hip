// rg_brick.hip -- hydro update of complete 8x8x8-oct bricks on gfx950.
//
// Paper Sec. 3 (the rock/paper kernels): larger blocks of octs share their
// stencil so that fewer ghost cells are reconstructed redundantly; the
// paper's "paper" kernel sweeps a planar stencil through the block.  Here a
// brick is a Hilbert-aligned cube of 8^3 octs (16^3 cells) that all exist at
// one level; because an aligned sub-cube is a contiguous stretch of the
// Hilbert order, its 512 octs are consecutive in memory.  One workgroup of
// four wavefronts marches through the brick plane by plane along z:
//   - thread t owns interior column (x, y) = (t % 16, t / 16) and keeps the
//     primitive variables of planes z-1, z, z+1 of that column in registers;
//   - the current plane's primitive variables, the face states and the face
//     fluxes are exchanged through LDS;
//   - the ghost ring of the plane (two cells wide) is shared by all columns,
//     so a cell is reconstructed once per brick instead of once per oct.
// The arithmetic is the same per-cell/per-face code as the per-oct kernel
// (rg_math.hpp), evaluated on the same operands in the same order, so the
// two kernels produce identical bits.
//
// Bricks are used only where every neighbour oct of the brick exists at the
// same level or lies outside the domain; octs of other bricks (touching a
// coarse ghost, or partial) go to the per-oct kernel.
#include "rg_internal.hpp"
#include "rg_math.hpp"
#include "rg_brick.hpp"

namespace rg {
namespace {

// Cost of n sweeps of nz planes with `slots` workgroups resident (`waves` per
// compute unit), in plane times of a full chip.  Measured on uniform boxes of
// 16^3 .. 256^3 cells over segments of 2 .. 256 planes: a sweep's two planes
// of ghost cells and its setup cost 2.6 (FP64) and 3.1 (mixed) planes; one
// workgroup per compute unit takes 3.4 us a plane in FP64 where two take 5.0
// us each, 2.5 us in the mixed form where two take 3.4 and three 4.3, so a
// round that leaves slots empty is that much quicker.
double sweep_cost(int64_t n, int nz, int slots, int waves)
{
    const int64_t full = n / slots, rest = n % slots;
    const double f = static_cast<double>(rest) / slots, one = 1.0 / waves;
    const double part = rest == 0 ? 0.0 : 0.35 + 0.65 * (f > one ? f : one);
    return (nz + 2.8) * (static_cast<double>(full) + part);
}

// Slabs that each of nbricks bricks is cut into: few bricks leave the chip
// empty and cost the whole latency of 16 planes (64 bricks: FP64 65 us whole,
// 26 us in four slabs; mixed 51 and 18 us in eight), many are best whole (512
// bricks: FP64 106 us whole, 121 in four slabs; mixed 75 and 77 us).
int brick_slabs(int64_t nbricks, int slots, int waves)
{
    int best = 1;
    for (int k = 2; k <= 8; k *= 2)
        if (sweep_cost(nbricks * k, BC / k, slots, waves) < sweep_cost(nbricks * best, BC / best, slots, waves))
            best = k;
    return best;
}

// Planes per segment of a column of `side` planes: 256^3, FP64 128 planes (512
// workgroups, one round of the chip; 694 us against 741 in 16-plane bricks),
// mixed 86 (768 workgroups; 504 against 536 us); 128^3, 16 (93 us) and 12 (62
// us); 32^3, 2 planes (15 us against 64 us for 8 whole bricks).
int column_planes(int64_t columns, int side, int slots, int waves)
{
    int best = side;
    double cost = sweep_cost(columns, side, slots, waves);
    for (int k = 2; k <= side / 2; ++k) {
        const int nz = ((side + k - 1) / k + 1) & ~1;
        const double c = sweep_cost(columns * ((side + nz - 1) / nz), nz, slots, waves);
        if (c < cost) {
            best = nz;
            cost = c;
        }
    }
    return best;
}

// W: waves per SIMD the register allocation is sized for (the compiler
// spills beyond it); KU: see brick_sweep.  FP64 keeps the state in registers
// at two waves; the mixed form keeps it at three (the default: no second
// read of uold, fewer bricks sharing an XCD's L2) or reads it again at four
// (with KU it would spill).  Every variant gives the same bits.
// Two face buffers (one barrier per plane less) where the LDS still holds
// as many workgroups as the registers allow: FP64 at two waves per SIMD
// (76 KB), mixed at four (40 KB: its partial updates then need no LDS
// slot) or three.
template <typename R, int W> constexpr int face_buffers() { return ((sizeof(R) == 8 && W == 2) || sizeof(R) == 4) ? 2 : 1; }

// Bricks of one or several levels, each cut into `slabs` of 16 / slabs planes.
template <typename R, int W, bool KU>
__global__ __launch_bounds__(BT, W) void k_hydro_brick(BrickArgs a, LevelTab lv, int slabs)
{
    __shared__ BrickSmem<R, face_buffers<R, W>()> S;
    // consecutive bricks on one XCD: workgroups are dealt round-robin to the
    // eight XCDs, so give each XCD a contiguous Hilbert range of bricks
    const int n = lv.item_end[lv.n - 1] * slabs;
    const int per_xcd = (n + 7) / 8;
    const int w = static_cast<int>(blockIdx.x % 8) * per_xcd + static_cast<int>(blockIdx.x / 8);
    if (w >= n) return;
    int b = w / slabs;
    const int nz = BC / slabs, z0 = (w - b * slabs) * nz;
    const int k = tab_entry(lv, b);
    a.dx = lv.dx[k];
    brick_body<R, KU>(a, a.bricks[lv.list0[k] + b], w, z0, nz, S);
}

// A complete level without split cells (the finest level of a uniform box) as
// columns of 16 x 16 cells, each cut into segments of nz planes.  Such a level
// needs no brick list: an oct's index is its place on the curve.  A longer
// sweep pays the two planes of ghost cells reconstructed at each end, and its
// setup, less often than a brick's 16 planes; the length is chosen by
// column_planes.  Columns in Morton order, each XCD a contiguous range with
// all its segments, so that neighbouring columns share their ghost cells in
// one L2.  Same operands, same order per cell: the same bits as bricks.
template <typename R, int W, bool KU>
__global__ __launch_bounds__(BT, W) void k_hydro_column(BrickArgs a, int nz)
{
    __shared__ BrickSmem<R, face_buffers<R, W>(), ColumnTable> S;
    const int side = 2 << a.nb;                   // cells per side
    const int nseg = (side + nz - 1) / nz;
    const int bits = a.nb - 3;                    // columns per side: 2^bits
    const int n = nseg << (2 * bits);
    const int per_xcd = (n + 7) / 8;
    const int w = static_cast<int>(blockIdx.x % 8) * per_xcd + static_cast<int>(blockIdx.x / 8);
    if (w >= n) return;
    const int col = w / nseg, z0 = (w - col * nseg) * nz;
    int bx = 0, by = 0;
    for (int t = 0; t < bits; ++t) {
        bx |= ((col >> (2 * t)) & 1) << t;
        by |= ((col >> (2 * t + 1)) & 1) << t;
    }
    column_body<R, KU>(a, BC * bx, BC * by, z0, min(nz, side - z0), w, S);
}

// workgroups resident per compute unit (four waves each), and on the chip
int wg_per_cu(int form, int waves) { return waves ? waves : (form == RG_FP64 ? 2 : 3); }

int wg_slots(int per_cu)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    return cus * per_cu;
}

BrickArgs brick_args(const rg_tree *t, const double *uold, double *unew, const int32_t *bricks, const double *dt,
                     double gamma, double cfl, double *dt_next, bool skip_split)
{
    BrickArgs a;
    a.skip_split = skip_split;
    a.uold = uold;
    a.unew = unew;
    a.nbr27 = t->d_nbr27;
    a.son = t->d_son_mask;
    a.keys = t->d_keys;
    a.bricks = bricks;
    a.dt = dt;
    a.dx = 0.0;
    a.gamma = gamma;
    a.outflow = t->bc == RG_BC_OUTFLOW;
    a.cfl = cfl;
    a.dt_next = reinterpret_cast<unsigned long long *>(dt_next);
    a.hdr = current_sink();
    a.first = 0;
    a.nb = 0;
    return a;
}

}  // namespace

rg_status hydro_bricks(const rg_tree *t, const double *uold, double *unew, const int32_t *list, const LevelTab &lv,
                       const double *dt, double gamma, int form, double cfl, double *dt_next, int waves,
                       bool skip_split, hipStream_t s)
{
    if (lv.n == 0) return RG_OK;
    const BrickArgs a = brick_args(t, uold, unew, list, dt, gamma, cfl, dt_next, skip_split);
    const int per_cu = wg_per_cu(form, waves);
    const int slabs = brick_slabs(tab_items(lv), wg_slots(per_cu), per_cu);
    const unsigned grid = static_cast<unsigned>(8 * ((tab_items(lv) * slabs + 7) / 8));
    if (form == RG_FP64) {
        if (waves == 0 || waves == 2)
            k_hydro_brick<double, 2, true><<<grid, BT, 0, s>>>(a, lv, slabs);
        else if (waves == 3)
            k_hydro_brick<double, 3, false><<<grid, BT, 0, s>>>(a, lv, slabs);
        else
            return fail(RG_ENOTSUP, "no FP64 brick kernel for %d waves per SIMD", waves);
    } else {
        if (waves == 4)
            k_hydro_brick<float, 4, false><<<grid, BT, 0, s>>>(a, lv, slabs);
        else if (waves == 0 || waves == 3)
            k_hydro_brick<float, 3, true><<<grid, BT, 0, s>>>(a, lv, slabs);
        else
            return fail(RG_ENOTSUP, "no mixed brick kernel for %d waves per SIMD", waves);
    }
    return launch_status("hydro bricks");
}

// complete level `level` (>= 4) without split cells
rg_status hydro_columns(const rg_tree *t, int level, const double *uold, double *unew, const double *dt, double gamma,
                        int form, double cfl, double *dt_next, int waves, hipStream_t s)
{
    BrickArgs a = brick_args(t, uold, unew, nullptr, dt, gamma, cfl, dt_next, false);
    a.dx = ldexp(1.0, -level);
    a.first = t->level_begin[level];
    a.nb = level - 1;
    const int64_t columns = int64_t(1) << (2 * (level - 4));
    const int per_cu = wg_per_cu(form, waves);
    const int nz = column_planes(columns, 1 << level, wg_slots(per_cu), per_cu);
    const int64_t n = columns * (((int64_t(1) << level) + nz - 1) / nz);
    const unsigned grid = static_cast<unsigned>(8 * ((n + 7) / 8));
    if (form == RG_FP64) {
        if (waves == 0 || waves == 2)
            k_hydro_column<double, 2, true><<<grid, BT, 0, s>>>(a, nz);
        else if (waves == 3)
            k_hydro_column<double, 3, false><<<grid, BT, 0, s>>>(a, nz);
        else
            return fail(RG_ENOTSUP, "no FP64 brick kernel for %d waves per SIMD", waves);
    } else {
        if (waves == 4)
            k_hydro_column<float, 4, false><<<grid, BT, 0, s>>>(a, nz);
        else if (waves == 0 || waves == 3)
            k_hydro_column<float, 3, true><<<grid, BT, 0, s>>>(a, nz);
        else
            return fail(RG_ENOTSUP, "no mixed brick kernel for %d waves per SIMD", waves);
    }
    return launch_status("hydro columns");
}

}  // namespace rg
