// Device re-tessellation of moved mesh points (section 2.1: the mesh is the
// Voronoi tessellation of its points, rebuilt after every move).
//
// Cell i of the new mesh is the set of points nearer to the new point r_i
// than to each candidate point, within the box for walls (its sides are the
// bisectors with the point's mirror images).  The candidates are the
// neighbours and the neighbours' neighbours of the cell in a previous mesh of
// the same points, each at its nearest periodic image (a periodic box of at
// least 16 cells, whose neighbours enclose each point).  The cell so found
// always contains the true Voronoi cell; it equals it when every true
// neighbour was a candidate.  The kernels certify that (every kept edge seen
// alike by both cells; the areas summing to the box area) instead of
// assuming it, and report failure so that the caller rebuilds on the host.
//
// No polygon is edited: each candidate's bisector is cut down to the part
// that every other candidate allows (two bounds kept as fractions), and the
// candidates with a non-empty part are the cell's edges; their parts' ends
// are the vertices.  The candidates (slots in LDS) are the wall mirrors and
// the previous neighbours; a neighbour's neighbour enters only when its
// bisector crosses the cell those give (one further than twice the largest
// vertex distance cannot, and is skipped at once).
//
// Most cells keep their neighbours from one step to the next; for those a
// cheaper proof suffices (k_rt_vertex: each vertex of the previous ring's
// consecutive neighbours checked against the other candidates), and the
// clip handles only the cells it leaves.
//
// Pipeline (one launch each, all on the caller's stream):
//   k_rt_begin    clear the result header and the queue counters, pack the
//                 new points in pairs
//   k_rt_vertex   a group of lanes per cell: the cell from its previous ring,
//                 when every vertex passes (else queued for the clip)
//   k_rt_near     (large meshes) the vertices against the neighbours' neighbours
//   k_rt_clip     a group of lanes per queued cell: the cell's edges, area,
//                 centroid
//   k_rt_count    kept and owned edges of each cell by the input stage's
//                 rules, scanned within blocks of cells
//   k_rt_scan_blocks  the scan over the blocks, totals, the checks of areas
//                 and capacities
//   k_rt_count_all  (small runs) both of these in one launch
//   k_rt_emit     off[], eoff[], edge records and the CSR entries of both
//                 sides of each edge, found in the neighbour's slots
//   k_rt_end      compares the few edges that emit cannot decide, folds the
//                 flags into the sticky word
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "rich.h"

namespace retess {

constexpr uint32_t kMask = 0x0FFFFFFFu;
constexpr int kShift = 28;
constexpr int kMaxFan = 20;    // edges of a finished cell (RICH_RETESS_FAN beyond)
static_assert(kMaxFan <= 64, "a kept slot's rank fits the six upper bits of its flag byte");
// Candidates of a cell besides the 4 mirrors of a walled box: neighbours in
// the previous mesh, and the neighbours' neighbours that entered.
constexpr int kSlots = 16;
// A cell's slots 0 .. kRow-1 lie in one 32-byte row, the rest (rare) apart.
constexpr int kRow = 8;
// deg[i] | kLean: a cell of at most kRow edges whose edges' lengths and
// midpoints follow from its row of neighbours to rounding far below what
// emit and end compare, every one of them kept (lean_cell); they are computed
// where they are needed instead of being stored and read back (24 bytes a
// slot).  On the 2048 x 2048 wave that is every cell; writing their geometry
// took the ring check from 371 to 666 us.
constexpr int32_t kLean = 1 << 8;
constexpr int kWallBits = 24;       // cnt of a lean cell, until counted: its walls from this bit on
constexpr int32_t kDegClip = -2;    // deg[i] of a cell that the ring check left to the clip,
constexpr int32_t kDegNear = -3;    // of one that the check of its neighbours' neighbours did
// The cells the vertex check leaves are queued for the clip in kSeg
// segments (block b of a run appends to segment b % kSeg), each with its own
// counter on its own 128-byte line, so that the blocks' appends do not all
// meet on one address; the clip's blocks then take them from there.
constexpr int kSeg = 64;
constexpr int kSegStride = 32;      // int32 counters 128 bytes apart
// A run of this many cells and more has the ring check and the check of the
// neighbours' neighbours as launches of their own, which loads less; below it
// one launch does both, and is the faster for it (a rebuild after moves of 0.02
// spacings, one launch against two: 55 and 71 us at 64 x 64 cells, 71 and 83 at
// 256 x 256, 115 and 107 at 362 x 362, 188 and 155 at 512 x 512, 668 and 477 at
// 1024 x 1024).  The run's own cells decide, not those of a batch together:
// the two forms send different cells to the clip (a neighbour's neighbour
// between the margins of two cells' tests), whose numbers are rounded
// otherwise, and a run's bits must not follow from its companions.  (By the
// cells of a whole batch 64 runs of 16 384 cells took 693 us, so 869; 6 of
// 65 536 262 and 313; 16 of 10 000 156 and 173.)
constexpr int kTieredMin = 98304;
// The two launches hand on the neighbours of the previous mesh's CSR entries
// in an array with room for those of a rebuilt mesh.  More entries (a previous
// mesh made by hand; none of Voronoi cells has more than 6 n + 2) take the one
// launch, by the entries in use: a mesh in large buffers names their room as
// its count, and then the kernels look at the last offset.
enum Form { kOneLaunch = 0, kTiered = 1, kByUse = 2 };
constexpr int kRingMax = 64;   // CSR entries read per cell of the previous mesh
constexpr int kThreads = 64;
constexpr int kScanThreads = 1024;
static_assert(kScanThreads % kThreads == 0, "a scan block covers whole cell blocks");
constexpr double kPi = 3.14159265358979323846;
// neighbour codes of the reflecting walls x = x0, x = x1, y = y0, y = y1 in
// the top bits of rich_edge.j (the neighbour is the cell's own mirror image)
constexpr int kWallX0 = 9, kWallX1 = 10, kWallY0 = 11, kWallY1 = 12;

struct Hdr {  // first 64 bytes of the workspace
  int32_t flags, sticky;
  int64_t n_edges, n_csr, n_dropped;
  double area_sum;
  int64_t n_wall;   // kept wall edges (each one CSR entry)
  int64_t n_clip;   // cells the vertex check left to the clip
  uint32_t done;    // blocks of k_rt_end that have finished (kUnlike: one found edges unlike)
  int32_t pad;
};
static_assert(sizeof(Hdr) == 64, "result header");

// One scan block's sums: area of its cells, dropped edge slots, kept wall
// edges.  Written per block and reduced in a fixed order by the scan, rather
// than added into the header with atomics (every block's atomics on one
// header line serialised the kernel).
struct CPart {
  double area;
  long long drop, walls, pad;
};

struct Args {
  // previous mesh (candidates)
  const int32_t* p_off;
  const int32_t* p_eoff;
  const int32_t* p_idx;
  const rich_edge* p_edges;
  int64_t p_n_csr, p_n_edges;
  // new points and output
  const double *x, *y;
  double2* xy;         // [n] the new points packed in pairs (filled by k_rt_begin)
  rich_cell* cells;
  rich_edge* edges;
  int32_t *off, *idx, *eoff;
  int64_t cap_edges, cap_csr;
  // workspace
  Hdr* hdr;
  int32_t* deg;        // [n] edges of the cell (| kLean), or a kDeg mark
  double* area;        // [n] the cells' areas, packed
  int32_t *s_nb, *s_nbx;   // [n][kRow], [n][kMaxFan - kRow] slots: cell | code << 28
  uint32_t* chk;       // [n] owned slots whose match with the neighbour's is still to compare
  // cells that are not lean only:
  double* s_geo;       // [n][kMaxFan][3] edge length, midpoint x, midpoint y
  uint8_t* s_flag;     // [n][kMaxFan] bit 0 kept, bit 1 owned, bits 2-6 rank among kept
  uint32_t* cnt;       // [n] kept | owned << 16 edges of a cell; then of its scan block before it
  int64_t* bsum;       // [2][n_scan_blocks] block totals of kept / owned
  CPart* cpart;        // [n_scan_blocks] block sums, reduced by the scan
  int32_t* qcnt;       // [kSeg * kSegStride] queue segment counters (every kSegStride-th)
  int32_t* queue;      // [kSeg][qcap] cells left to the clip
  int32_t* nb;         // [nb_cap] neighbour of each CSR entry of the previous mesh
  int64_t nb_cap;
  int64_t nb_end;      // entries that have a place there: min(p_n_csr, nb_cap)
  int32_t* flag_out;   // if set, the flags also go here, and the counts to info_out
  rich_retess_info* info_out;
  int32_t qcap;        // capacity of a segment: kThreads * ceil(cell blocks / kSeg)
  // geometry
  double x0, y0, x1, y1, Lx, Ly;
  double size;         // largest of the box's sides and its corners' coordinates
  int32_t n, bc, n_scan_blocks, form;
};

// Many runs in one launch: run r's descriptor is descs[r]; its blocks of
// kThreads cells are cstart[r] .. cstart[r+1]-1 and its scan blocks of
// kScanThreads cells sstart[r] .. sstart[r+1]-1; hdr_out[r] receives its
// result header at the end.
struct Batch {
  const Args* descs;
  const int32_t* cstart;
  const int32_t* sstart;
  Hdr* hdr_out;
  int32_t* flags_out;   // each run's flags, for rich_retess_batch_flags_async
  int32_t n_runs;
};

// Run of block b in a start table of n_runs + 1 entries.
__device__ __forceinline__ int run_of_block(const int32_t* __restrict__ start, int n_runs, int b) {
  int lo = 0, hi = n_runs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The descriptor of the run of block b of a launch and the block's index
// within the run.
template <bool B>
__device__ __forceinline__ const Args& block_run(const Args& one, const int32_t* start,
                                                 const Batch& bt, int b, int& blk) {
  if (!B) {
    blk = b;
    return one;
  }
  const int r = run_of_block(start, bt.n_runs, b);
  blk = b - start[r];
  return bt.descs[r];
}
// Whether the run has the two launches (Form).
__device__ __forceinline__ bool tiered(const Args& a) {
  return a.form == kTiered || (a.form == kByUse && a.p_off[a.n] <= a.nb_cap);
}
// The block of cells this block works on: each of the 8 XCDs (with an L2 of
// its own, taking every eighth block of a launch) gets one contiguous range
// of them, so that the neighbours' rows, points and offsets that a block
// gathers are mostly in its XCD's L2 (2048 x 2048 wave, read from beyond it
// with plain order and with this: ring check 0.87 and 0.60 GB, near check 0.37
// and 0.18, emit 0.49 and 0.24; 511 x 511 tube, emit: 19.8 -> 18.6 us).
__device__ __forceinline__ int cell_block() {
  constexpr int kNumXcd = 8;
  const int nb = gridDim.x, x = blockIdx.x % kNumXcd, rem = nb % kNumXcd;
  return x * (nb / kNumXcd) + min(x, rem) + blockIdx.x / kNumXcd;
}

__device__ __forceinline__ int32_t pack(int cell, int code) {
  return (int32_t)((uint32_t)cell | ((uint32_t)code << kShift));
}
// periodic image shift (sx, sy) in box lengths <-> code 1..8 (0 is no shift)
__device__ __forceinline__ int shift_code(int sx, int sy) {
  const int k = (sx + 1) * 3 + (sy + 1);
  return k < 4 ? k + 1 : k;
}
__device__ __forceinline__ void code_shift(int code, int& sx, int& sy) {
  const int k = code <= 4 ? code - 1 : code;
  sx = k / 3 - 1;
  sy = k % 3 - 1;
}
__device__ __forceinline__ int back_code(int code) { return code == 0 ? 0 : 9 - code; }

// The point p with p.a = |a|^2/2 and p.b = |b|^2/2 (the Voronoi vertex of the
// origin and the points a and b); false unless b is counter-clockwise of a.
__device__ __forceinline__ bool bisector_meet(double ax, double ay, double bx, double by,
                                              double& px, double& py) {
  const double det = ax * by - ay * bx;
  const double ha = 0.5 * (ax * ax + ay * ay), hb = 0.5 * (bx * bx + by * by);
  px = (ha * by - hb * ay) / det;
  py = (ax * hb - ha * bx) / det;
  return det > 0.0;
}

// Neighbour cell that a CSR entry of the previous mesh names (-1 if out of
// range); of CSR entry k.
__device__ __forceinline__ int entry_cell(const Args& a, int ent) {
  const int e = ent >> 1;
  if (ent < 0 || e >= a.p_n_edges) return -1;
  const int2 ij = *reinterpret_cast<const int2*>(&a.p_edges[e].i);
  return (ent & 1) ? ij.x : (int)((uint32_t)ij.y & kMask);
}
__device__ __forceinline__ int prev_neighbour(const Args& a, int k) {
  return entry_cell(a, a.p_idx[k]);
}

// Clears the result header and the queue counters (each run's first block)
// and packs the new points in pairs, so that a candidate's point is one
// 16-byte load (the kernels gather them by cell index many times over).
template <bool B>
__global__ __launch_bounds__(kThreads) void k_rt_begin(Args one, Batch bt) {
  int blk;
  const Args& a = block_run<B>(one, bt.cstart, bt, cell_block(), blk);
  if (blk == 0) {
    Hdr* h = a.hdr;
    for (int t = threadIdx.x; t < kSeg; t += kThreads) a.qcnt[t * kSegStride] = 0;
    if (threadIdx.x == 0) {
      h->flags = 0;
      h->n_edges = 0;
      h->n_csr = 0;
      h->n_dropped = 0;
      h->area_sum = 0.0;
      h->n_wall = 0;
      h->n_clip = 0;
      h->done = 0;
    }
  }
  const int i = blk * kThreads + threadIdx.x;
  if (i < a.n) a.xy[i] = make_double2(a.x[i], a.y[i]);
}

// ---------------------------------------------------------------------------
// groups of lanes
// ---------------------------------------------------------------------------
// kGroup lanes work on a cell: one per neighbour, candidate or slot.
constexpr int kGroup = 8;               // lanes (and ring entries) of a cell
constexpr int kGroupThreads = kThreads * kGroup;
static_assert(64 % kGroup == 0, "groups do not straddle waves");

// The group's bits of a wave-wide ballot.
__device__ __forceinline__ uint32_t group_bits(bool v) {
  const unsigned long long m = __ballot(v);
  const int first = (int)(threadIdx.x & 63) & ~(kGroup - 1);
  return (uint32_t)(m >> first) & ((1u << kGroup) - 1u);
}
// The value of the lane opposite in the group at distance 1, 2 (quad
// permutations) or in the other quad (half-row mirror, of values equal
// within a quad): moves on the vector ALU.
template <int CTRL>
__device__ __forceinline__ double dpp_of(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true),
                          __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141;
// Larger of two doubles by the instruction alone (fmax first quiets operands
// that the compiler cannot prove quiet; none here is a signalling NaN).
__device__ __forceinline__ double dmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double group_max(double v) {
  v = dmax(v, dpp_of<kDppXor1>(v));
  v = dmax(v, dpp_of<kDppXor2>(v));
  return dmax(v, dpp_of<kDppHalfMirror>(v));
}
__device__ __forceinline__ double group_sum(double v) {
  v += dpp_of<kDppXor1>(v);
  v += dpp_of<kDppXor2>(v);
  return v + dpp_of<kDppHalfMirror>(v);
}

__device__ __forceinline__ uint32_t group_or(uint32_t v) {
  v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor1, 0xF, 0xF, true);
  v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor2, 0xF, 0xF, true);
  return v | (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppHalfMirror, 0xF, 0xF, true);
}
__device__ __forceinline__ int group_or(int v) { return (int)group_or((uint32_t)v); }
// The lanes of one wave read what others of it wrote.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// Displacement of point (xc, yc) of cell c from (xi, yi) (nearest periodic
// image) and its id.  The image is sought only when some lane of the wave
// needs it (a wave holds nearby cells, so all but the waves at the box's
// edges skip it); otherwise the plain difference is that image, of code 0.
template <bool WALLS>
__device__ __forceinline__ int32_t displacement(const Args& a, double xi, double yi, int c,
                                                double xc, double yc, double& dx, double& dy) {
  dx = xc - xi;
  dy = yc - yi;
  int code = 0;
  if (!WALLS && __any(fabs(dx) > 0.5 * a.Lx || fabs(dy) > 0.5 * a.Ly)) {
    int sx = 0, sy = 0;
    if (dx > 0.5 * a.Lx) { dx -= a.Lx; sx = -1; } else if (dx < -0.5 * a.Lx) { dx += a.Lx; sx = 1; }
    if (dy > 0.5 * a.Ly) { dy -= a.Ly; sy = -1; } else if (dy < -0.5 * a.Ly) { dy += a.Ly; sy = 1; }
    if (sx != 0 || sy != 0) code = shift_code(sx, sy);
  }
  return pack(c, code);
}

// ---------------------------------------------------------------------------
// the cell of one point
// ---------------------------------------------------------------------------
// Counter-clockwise order of directions: the upper half-plane (from angle 0
// inclusive) before the lower one, then by the sign of the cross product.
__device__ __forceinline__ bool ccw_before(double ax, double ay, double bx, double by) {
  const int ha = (ay < 0.0 || (ay == 0.0 && ax < 0.0)) ? 1 : 0;
  const int hb = (by < 0.0 || (by == 0.0 && bx < 0.0)) ? 1 : 0;
  if (ha != hb) return ha < hb;
  return ax * by - ay * bx > 0.0;
}

// The part of the bisector of displacement (dux, duy) (the line
// p.d = |d|^2/2, parametrised p(t) = d/2 + t (-duy, dux), t increasing
// counter-clockwise about r_i) that satisfies p.d_v <= |d_v|^2/2 for every
// candidate v it was cut by: [lo, hi].  The bounds are kept as fractions and
// compared by cross-multiplication, so a cut divides nothing, and no bound
// yet is hn / hd = +inf and ln / ld = -inf: the first finite bound of each
// side then wins its comparison (b and a are finite), so no flag tracks
// whether a side is bounded.
struct Part {
  double mux, muy, eux, euy;
  double ln = -INFINITY, ld = 1.0, hn = INFINITY, hd = 1.0;
  bool empty = false;
  __device__ Part(double dux, double duy)
      : mux(0.5 * dux), muy(0.5 * duy), eux(-duy), euy(dux) {}
  // straight-line (selects, no branches)
  // (dvh: half of the displacement's square)
  __device__ __forceinline__ void cut(double dvx, double dvy, double dvh, bool act) {
    const double a = eux * dvx + euy * dvy;
    const double b = dvh - (mux * dvx + muy * dvy);
    // a > 0: t <= b / a;  a < 0: t >= (-b) / (-a);  a = 0, b < 0: no t
    const bool up = act && a > 0.0 && b * hd < hn * a;
    hn = up ? b : hn;
    hd = up ? a : hd;
    const bool dn = act && a < 0.0 && -b * ld > ln * -a;
    ln = dn ? -b : ln;
    ld = dn ? -a : ld;
    empty = empty || (act && a == 0.0 && b < 0.0);
  }
  // false when one end is open (the candidates do not enclose the point)
  __device__ __forceinline__ bool bounded() const { return ln != -INFINITY && hn != INFINITY; }
  __device__ __forceinline__ bool live() const { return !empty && bounded() && ln * hd < hn * ld; }
};

// The vertex equidistant from r_i and the points at displacements a and b, b
// counter-clockwise after a by less than half a turn (det = |a| |b| sin(angle),
// by a margin); false if it is not.
constexpr double kVertexSin = 0.05;     // least sine of a consecutive pair's angle
constexpr double kVertexMargin = 1e-9;  // relative margin of every vertex test
__device__ __forceinline__ bool ring_vertex(double ax, double ay, double bx, double by,
                                            double& vx, double& vy) {
  const double ha = 0.5 * (ax * ax + ay * ay), hb = 0.5 * (bx * bx + by * by);
  const double det = ax * by - ay * bx;
  const bool turn = det > 0.0 && det * det > (4.0 * kVertexSin * kVertexSin) * ha * hb;
  const double inv = 1.0 / (turn ? det : 1.0);
  vx = (ha * by - hb * ay) * inv;
  vy = (ax * hb - ha * bx) * inv;
  return turn;
}
// Length and midpoint of the edge from vertex u to vertex w about (xi, yi).
__device__ __forceinline__ void edge_geometry(double xi, double yi, double ux, double uy, double wx,
                                              double wy, double& len, double& mx, double& my) {
  const double ex = wx - ux, ey = wy - uy;
  len = sqrt(ex * ex + ey * ey);
  mx = xi + 0.5 * (ux + wx);
  my = yi + 0.5 * (uy + wy);
}
// Displacement of the point that slot `id` of the cell at (xi, yi) names (p
// its cell's, or for a wall the cell's own).
__device__ __forceinline__ void slot_displacement(const Args& a, double xi, double yi, int32_t id,
                                                  double2 p, double& dx, double& dy) {
  dx = p.x - xi;
  dy = p.y - yi;
  const int code = (int)((uint32_t)id >> kShift);
  if (code >= kWallX0) {   // the mirror image
    dx = code == kWallX0 ? 2.0 * (a.x0 - xi) : code == kWallX1 ? 2.0 * (a.x1 - xi) : 0.0;
    dy = code == kWallY0 ? 2.0 * (a.y0 - yi) : code == kWallY1 ? 2.0 * (a.y1 - yi) : 0.0;
  } else if (code != 0) {
    int sx, sy;
    code_shift(code, sx, sy);
    dx += sx * a.Lx;
    dy += sy * a.Ly;
  }
}
// Whether a cell whose consecutive neighbours all turn by ring_vertex's
// margin is lean: its shortest edge (squared length l2) is above the cut for
// dropping one whatever the neighbour's area (2e-12 box radii); and rounding,
// of the vertices (about 1e-14 of the largest distance, squared r2) and of the
// coordinates (4e-15 of their size a.size), stays below half of the
// tolerance of k_rt_end's comparison, 1e-9 cell radii.
__device__ __forceinline__ bool lean_cell(const Args& a, double l2, double r2, double area) {
  return l2 >= 4e-24 / kPi * a.Lx * a.Ly && r2 <= 3e5 * area && area >= 2e-10 * a.size * a.size;
}
__device__ __forceinline__ int32_t& slot_nb(const Args& a, int i, int q) {
  return q < kRow ? a.s_nb[(size_t)i * kRow + q]
                  : a.s_nbx[(size_t)i * (kMaxFan - kRow) + (q - kRow)];
}

// The cells of a queue, kGroup lanes each: lane l holds candidates l, l +
// kGroup, ..., so the trials of every candidate against every other one, a
// serial chain of hundreds of operations and loads for one lane, run side by
// side, and lane l goes through the row of ring member l.  A neighbour's
// neighbour is first tried against the vertices of the polygon that the ring
// gives (three operations a vertex, four candidates at a time); only the few
// that may cut it meet the trial against every candidate.  A small mesh queues
// a wave or two of cells, and the chain on an otherwise idle chip is its time:
// one lane per cell took 143 us for 600 cells of a 64 x 64 tube, 16 lanes 33,
// this 20; of 60 113 cells of a 511 x 511 one 205, 111 and 51 us; of 370 000
// cells (2048 x 2048 wave), where the vector ALU is the bound, 16 lanes without
// that first trial took 465 us (2000 instructions for 4 cells), this 247.  (One
// candidate at a time: 25, 66 and 305 us.)
constexpr int kClipThreads = 256;
constexpr int kClipCells = kClipThreads / kGroup;   // cells of a block at a time
constexpr int kClipMaxBlocks = kSeg * 32;           // of one run: the blocks stride

// A cell's candidates in LDS, read by the whole group: displacement from r_i
// to the generating point, half its square, id (cell | code << 28); the
// vertices of the ring's polygon; the slot of the edge at each place.  (The
// size, 16 bytes past a multiple of 256, keeps the groups of a wave on
// different banks.)
template <int NS>
struct ClipSlots {
  double2 v[NS];
  double dx[NS], dy[NS], h[NS];
  int32_t id[NS], place[NS];
  static constexpr size_t kBytes = NS * (16 + 24 + 4 + 4);
  char pad[(kBytes + 239) / 256 * 256 + 16 - kBytes];
};
static_assert(sizeof(ClipSlots<16>) == 784 && sizeof(ClipSlots<20>) == 1040, "banks");

// One queued cell.  With walls, the first slots hold the point's mirrors (they
// bound it), without those far beyond the ring if the ring bounds it closer;
// then come the cell's neighbours in the previous mesh; the first pass finds
// the polygon those allow.  The neighbours' neighbours then enter
// only when their bisector crosses that polygon; the second pass gives the
// cell, its area, centroid and edges in counter-clockwise order.  (TIERED:
// the neighbours are read where the ring check wrote them.)
template <bool WALLS, bool TIERED>
__device__ void clip_cell(const Args& a, int i, ClipSlots<kSlots + (WALLS ? 4 : 0)>& S) {
  constexpr int NS = kSlots + (WALLS ? 4 : 0);    // candidates per cell
  constexpr int H = (NS + kGroup - 1) / kGroup;   // of each lane
  constexpr int RH = kSlots / kGroup;   // ring members of each lane
  static_assert(NS <= kMaxFan && kSlots % kGroup == 0, "slots");
  const int l = (int)threadIdx.x & (kGroup - 1);
  const double xi = a.x[i], yi = a.y[i];
  int bad = 0;
  auto put_slot = [&](int u, double dx, double dy, int32_t id) {
    S.dx[u] = dx;
    S.dy[u] = dy;
    S.h[u] = 0.5 * (dx * dx + dy * dy);
    S.id[u] = id;
  };
  if (WALLS) {
    if (!(xi > a.x0 && xi < a.x1 && yi > a.y0 && yi < a.y1)) bad |= RICH_RETESS_POINT;
  } else {
    // no bounds: the neighbours enclose the point (a cell they leave open
    // is reported, and rebuilt on the host)
    if (!(xi >= a.x0 && xi < a.x1 && yi >= a.y0 && yi < a.y1)) bad |= RICH_RETESS_POINT;
  }

  // the ring: lane l loads CSR entries l and l + kGroup (-1: past the end,
  // out of range, or the cell itself, as a wall's entry is)
  int k0 = 0, k1 = 0;
  if (!bad) {
    k0 = a.p_off[i];
    k1 = a.p_off[i + 1];
    if (k0 < 0 || k1 < k0 || k1 > (TIERED ? a.nb_end : a.p_n_csr)) {
      bad |= RICH_RETESS_CLIP;
      k1 = k0;
    } else if (k1 - k0 > kSlots) {
      bad |= RICH_RETESS_FAN;
      k1 = k0;
    }
  }
  int c[RH];
#pragma unroll
  for (int h = 0; h < RH; ++h) {
    const int k = k0 + l + h * kGroup;
    c[h] = k < k1 ? (TIERED ? a.nb[k] : prev_neighbour(a, k)) : -1;
    if (c[h] >= a.n || c[h] == i) c[h] = -1;
  }
  double rx[RH], ry[RH], far2 = 0.0;
  int32_t rid[RH];
  int row0[RH], row1[RH];   // the ring members' rows (of no member: none)
#pragma unroll
  for (int h = 0; h < RH; ++h) {
    row0[h] = c[h] < 0 ? 0 : a.p_off[c[h]];
    row1[h] = c[h] < 0 ? 0 : a.p_off[c[h] + 1];
    const double2 p = a.xy[c[h] < 0 ? i : c[h]];
    rid[h] = displacement<WALLS>(a, xi, yi, c[h], p.x, p.y, rx[h], ry[h]);
    far2 = fmax(far2, rx[h] * rx[h] + ry[h] * ry[h]);
  }
  // lane l < 4: the point's mirror across the walls y0, x1, y1, x0
  double wx = 0.0, wy = 0.0;
  bool mirror = false;
  if (WALLS) {
    wx = l == 1 ? 2.0 * (a.x1 - xi) : (l == 3 ? 2.0 * (a.x0 - xi) : 0.0);
    wy = l == 0 ? 2.0 * (a.y0 - yi) : (l == 2 ? 2.0 * (a.y1 - yi) : 0.0);
    // One cuts the ring's polygon only from within twice its largest vertex
    // distance, about 0.7 of the farthest neighbour's: those within 1.4 of that
    // are taken at first (within 2: a step of 4096 cells 134.7 us, so 130.5).
    // (A move reads nothing from a lane that a branch has switched off, so all
    // lanes take the maximum, before the && below.)
    const double near2 = 2.0 * group_max(far2);
    mirror = l < 4 && wx * wx + wy * wy <= near2;
  }

  // first pass: the polygon of the bounds and the first ring, and the
  // largest distance of its vertices
  int base, nv;   // mirror slots; slots
  uint32_t em;
  double reach2;
  for (;;) {
    base = 0;
    if (WALLS) {
      const uint32_t in = group_bits(mirror);
      if (mirror)
        put_slot(__popc(in & ((1u << l) - 1u)), wx, wy,
                 pack(i, l == 0 ? kWallY0 : l == 1 ? kWallX1 : l == 2 ? kWallY1 : kWallX0));
      base = __popc(in);
    }
    nv = base;
#pragma unroll
    for (int h = 0; h < RH; ++h) {
      const uint32_t in = group_bits(c[h] >= 0);
      if (c[h] >= 0) put_slot(nv + __popc(in & ((1u << l) - 1u)), rx[h], ry[h], rid[h]);
      nv += __popc(in);
    }
    wave_sync();
    em = 0;
    reach2 = 0.0;
    int open = 0;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int u = l + h * kGroup;
      bool live = false;
      double px = 0.0, py = 0.0;
      if (!bad && u < nv) {
        const double dux = S.dx[u], duy = S.dy[u];
        const int32_t idu = S.id[u];
        Part p(dux, duy);
#pragma unroll 2
        for (int v = 0; v < nv; ++v) {
          const bool same = v != u && S.id[v] == idu;   // a duplicate: the first stands
          p.empty = p.empty || (same && v < u);
          p.cut(S.dx[v], S.dy[v], S.h[v], v != u && !same);
        }
        live = p.live();
        if (live) {
          const double t = p.hn / p.hd;
          px = 0.5 * dux - t * duy;
          py = 0.5 * duy + t * dux;
          reach2 = fmax(reach2, px * px + py * py);
        } else if (!p.bounded()) {
          open = RICH_RETESS_CLIP;
        }
      }
      const uint32_t lv = group_bits(live);
      if (live) S.v[__popc(em) + __popc(lv & ((1u << l) - 1u))] = make_double2(px, py);
      em |= lv << (h * kGroup);
    }
    reach2 = group_max(reach2);
    open = group_or(open);
    wave_sync();
    // a mirror left out that may cut the polygon, or one to bound it: all in
    if (WALLS && base < 4 &&
        (open != 0 || em == 0u ||
         group_bits(l < 4 && !mirror && !(4.0 * reach2 <= wx * wx + wy * wy)) != 0u)) {
      mirror = l < 4;
      continue;
    }
    bad |= open;
    break;
  }
  const int corners = __popc(em);

  // the neighbours' neighbours, lane l through the row of ring member l: those
  // that are new and may cut the polygon (one further than twice its largest
  // vertex distance cannot, nor one whose half plane holds every vertex by the
  // margin) meet the full trial, each lane's first, then its second, ...  One
  // enters when its bisector crosses the polygon of the slots, which includes
  // those that entered before it: the lanes try theirs against the slots
  // together, and those that cross then enter in order, each one cutting the
  // ones after it.
  const double mr = kVertexMargin * reach2;
#pragma unroll 1
  for (int h = 0; h < RH && !bad; ++h) {
    const int cm = h == 0 ? c[0] : c[RH - 1];
    static_assert(RH == 2, "two ring members of a lane");
    int k = h == 0 ? row0[0] : row0[RH - 1], k1 = h == 0 ? row1[0] : row1[RH - 1];
    if (cm >= 0) {
      if (k < 0 || k1 < k || k1 > (TIERED ? a.nb_end : a.p_n_csr) || k1 - k > kRingMax) {
        bad = RICH_RETESS_CLIP;
        k1 = k;
      }
    }
    bad = group_or(bad);
    constexpr int CH = 8;   // candidates of a lane whose loads are in flight together
    constexpr int QD = 4;   // ... that one read of a slot or a vertex is tried on
    for (; group_bits(k < k1) != 0u && !bad; k += CH) {
      uint32_t may = 0;   // the chunk's candidates for the full trial
      int cc[CH];
      double2 cp[CH];
      const int tried = nv;   // slots that they are compared with here
#pragma unroll
      for (int t = 0; t < CH; ++t)
        cc[t] = k + t < k1 ? (TIERED ? a.nb[k + t] : a.p_idx[k + t]) : -1;
      if (!TIERED) {
#pragma unroll
        for (int t = 0; t < CH; ++t) cc[t] = entry_cell(a, cc[t]);
      }
#pragma unroll
      for (int t = 0; t < CH; ++t) {
        if (cc[t] >= a.n || cc[t] == i) cc[t] = -1;
        cp[t] = a.xy[cc[t] < 0 ? 0 : cc[t]];
      }
#pragma unroll
      for (int g = 0; g < CH; g += QD) {
        double dx[QD], dy[QD], q[QD];   // q: the largest projection of a vertex
        int32_t id[QD];
        bool on[QD], any = false;
#pragma unroll
        for (int t = 0; t < QD; ++t) {
          id[t] = displacement<WALLS>(a, xi, yi, cc[g + t], cp[g + t].x, cp[g + t].y, dx[t], dy[t]);
          on[t] = cc[g + t] >= 0 && !(4.0 * reach2 <= dx[t] * dx[t] + dy[t] * dy[t]);
          q[t] = -INFINITY;
          any = any || on[t];
        }
        if (!any) continue;
        for (int v = base; v < nv; ++v) {
          const int32_t idv = S.id[v];
#pragma unroll
          for (int t = 0; t < QD; ++t) on[t] = on[t] && idv != id[t];
        }
        for (int v = 0; v < corners; ++v) {
          const double2 pv = S.v[v];
#pragma unroll
          for (int t = 0; t < QD; ++t) q[t] = dmax(q[t], pv.x * dx[t] + pv.y * dy[t]);
        }
#pragma unroll
        for (int t = 0; t < QD; ++t) {
          const double hu = 0.5 * (dx[t] * dx[t] + dy[t] * dy[t]);
          if (on[t] && !(hu - q[t] > kVertexMargin * hu + mr)) may |= 1u << (g + t);
        }
      }
      for (; group_bits(may != 0u) != 0u && !bad; may &= may - 1u) {
        bool on = may != 0u;
        const int tt = on ? __ffs(may) - 1 : 0;
        int cj = i;
        double2 pj = make_double2(xi, yi);
        if (TIERED) {   // (kept in registers, they would cost a wave per SIMD)
          if (on) cj = a.nb[k + tt];   // (in range: tried)
          pj = a.xy[cj];
        } else {
#pragma unroll
          for (int t = 0; t < CH; ++t) {
            if (on && t == tt) {
              cj = cc[t];
              pj = cp[t];
            }
          }
        }
        double dx, dy;
        const int32_t id = displacement<WALLS>(a, xi, yi, cj, pj.x, pj.y, dx, dy);
        // those that entered since (in a full list they may have any place)
        for (int v = nv < NS ? tried : base; v < nv; ++v) on = on && S.id[v] != id;
        if (group_bits(on) == 0u) continue;
        Part p(dx, dy);
#pragma unroll 2
        for (int v = 0; v < nv; ++v) p.cut(S.dx[v], S.dy[v], S.h[v], true);
        uint32_t in;
        while ((in = group_bits(on && p.live())) != 0u && !bad) {
          const int f = __ffs(in) - 1;
          // a new slot, else one whose bisector bounds nothing (it stays
          // redundant as candidates are added; a mirror is never reused)
          int u = nv;
          if (nv < NS) {
            ++nv;
          } else {
            const uint32_t usable = ~em & ((1u << NS) - 1u) & ~((1u << base) - 1u);
            u = __ffs(usable) - 1;
            if (usable == 0u) {
              bad = RICH_RETESS_FAN;
              break;
            }
          }
          em |= 1u << u;   // holds a cutting candidate now: not reusable
          wave_sync();
          if (l == f) put_slot(u, dx, dy, id);
          wave_sync();
          on = on && id != S.id[u];
          p.cut(S.dx[u], S.dy[u], S.h[u], on);
        }
      }
    }
  }

  rich_cell cr;
  cr.px = xi;
  cr.py = yi;
  cr.pad = 0.0;
  cr.area = 0.0;
  cr.sx = xi;
  cr.sy = yi;
  // second pass: each candidate's part of its bisector.  A live one is an
  // edge: its place is its counter-clockwise rank among all the candidates
  // (the upper half-plane, from angle 0 inclusive, before the lower one, then
  // by the sign of the cross product, then by slot) less the ranks of those
  // that bound nothing.
  uint32_t lower = 0;   // slots in the lower half-plane
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int u = l + h * kGroup;
    const double dx = u < nv ? S.dx[u] : 0.0, dy = u < nv ? S.dy[u] : 0.0;
    lower |= group_bits(dy < 0.0 || (dy == 0.0 && dx < 0.0)) << (h * kGroup);
  }
  uint32_t fm = 0, holes = 0;
  int rank[H];
  double len_[H], mx[H], my[H];
  double A2 = 0.0, cx = 0.0, cy = 0.0, l2 = INFINITY;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int u = l + h * kGroup;
    bool live = false;
    rank[h] = 0;
    len_[h] = mx[h] = my[h] = 0.0;
    if (!bad && u < nv) {
      const double dux = S.dx[u], duy = S.dy[u];
      const int32_t idu = S.id[u];
      const bool low = (lower >> u) & 1u;
      Part p(dux, duy);
#pragma unroll 2
      for (int v = 0; v < nv; ++v) {
        const double dvx = S.dx[v], dvy = S.dy[v];
        const bool other = v != u;
        const bool same = other && S.id[v] == idu;
        p.empty = p.empty || (same && v < u);
        p.cut(dvx, dvy, S.h[v], other && !same);
        // (two products, each rounded: the sign is the opposite one from v's side)
        const double r = dvx * duy;
        const double s = dvy * dux;
        const bool lowv = (lower >> v) & 1u;
        rank[h] += other && (lowv == low ? r > s || (r == s && v < u) : low) ? 1 : 0;
      }
      live = p.live();
      if (live) {
        const double tlo = p.ln / p.ld, thi = p.hn / p.hd;
        const double ux = 0.5 * dux - tlo * duy, uy = 0.5 * duy + tlo * dux;
        const double wx = 0.5 * dux - thi * duy, wy = 0.5 * duy + thi * dux;
        const double cv = ux * wy - uy * wx;
        A2 += cv;
        cx += (ux + wx) * cv;
        cy += (uy + wy) * cv;
        edge_geometry(xi, yi, ux, uy, wx, wy, len_[h], mx[h], my[h]);
        l2 = fmin(l2, len_[h] * len_[h]);
      } else {
        if (!p.bounded()) bad |= RICH_RETESS_CLIP;
        holes |= 1u << rank[h];
      }
    }
    fm |= group_bits(live) << (h * kGroup);
  }
  holes = group_or(holes);
  bad = group_or(bad);
  A2 = group_sum(A2);
  cx = group_sum(cx);
  cy = group_sum(cy);
  const int deg = __popc(fm);
  if (deg < 3) bad |= RICH_RETESS_CLIP;
  // the edges' places; rounding that ranks two of them alike fails the cell
  int q[H];
  uint32_t taken = 0;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    q[h] = (fm >> (l + h * kGroup)) & 1u ? rank[h] - __popc(holes & ((1u << rank[h]) - 1u))
                                         : kMaxFan;   // (a place is < NS <= kMaxFan)
    taken |= 1u << q[h];
  }
  taken = group_or(taken);
  if ((taken & ((1u << kMaxFan) - 1u)) != (1u << deg) - 1u) bad |= RICH_RETESS_CLIP;
  if (bad) {
    if (l == 0) {
      atomicOr(&a.hdr->flags, bad);
      a.deg[i] = 0;
      a.area[i] = 0.0;
      a.cells[i] = cr;
    }
    return;
  }
  bool wall = false;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (q[h] < kMaxFan) {
      const int u = l + h * kGroup;
      slot_nb(a, i, q[h]) = S.id[u];
      S.place[q[h]] = u;   // (all of 0 .. deg - 1 are taken)
    }
  }
  wave_sync();
  // lean if every consecutive pair turns enough, and the rest of lean_cell
  double r2 = 0.0;
  bool plain = deg <= kRow, own = false;
  static_assert(kRow == kGroup, "a lane per slot of a row");
  if (plain && l < deg) {
    const int u = S.place[l], v = S.place[l + 1 < deg ? l + 1 : 0];
    double vx, vy;
    plain = ring_vertex(S.dx[u], S.dy[u], S.dx[v], S.dy[v], vx, vy);
    r2 = vx * vx + vy * vy;
    wall = (int)((uint32_t)S.id[u] >> kShift) >= kWallX0;
    own = wall || i < (int)((uint32_t)S.id[u] & kMask);
  }
  r2 = group_max(r2);
  l2 = -group_max(-l2);
  const bool lean = group_bits(!plain) == 0u && lean_cell(a, l2, r2, 0.5 * A2);
  const uint32_t owns = group_bits(own), walls = group_bits(wall);
  if (!lean) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (q[h] < kMaxFan) {
        double* g = a.s_geo + 3 * ((size_t)i * kMaxFan + q[h]);
        g[0] = len_[h];
        g[1] = mx[h];
        g[2] = my[h];
      }
    }
  }
  if (l == 0) {
    a.deg[i] = deg | (lean ? kLean : 0);
    // (if lean: deg <= kRow)
    a.cnt[i] = (uint32_t)deg | (uint32_t)__popc(owns) << 16 | (uint32_t)__popc(walls) << kWallBits;
    a.area[i] = 0.5 * A2;
    cr.area = 0.5 * A2;
    cr.sx = xi + cx / (3.0 * A2);
    cr.sy = yi + cy / (3.0 * A2);
    a.cells[i] = cr;
  }
}

// Block b of a run takes entries of queue segment b % kSeg, as many cells at
// a time as it has groups.  Each launch serves one kind of run (a batch of
// both kinds takes two launches), so a run's results never depend on the
// other runs.
template <bool B, bool WALLS, bool TIERED>
__global__ __launch_bounds__(kClipThreads) void k_rt_clip(Args one, Batch bt) {
  __shared__ ClipSlots<kSlots + (WALLS ? 4 : 0)> s_slots[kClipCells];
  int blk, nblk = gridDim.x;
  const Args& a = block_run<B>(one, bt.cstart, bt, blockIdx.x, blk);
  if ((a.bc == (int)RICH_BOUNDARY_PERIODIC) == WALLS || tiered(a) != TIERED)
    return;  // another launch's run
  if (B) nblk = (a.n + kThreads - 1) / kThreads;
  const int seg = blk % kSeg;
  const int queued = min(a.qcnt[seg * kSegStride], a.qcap);
  const int group = (int)threadIdx.x / kGroup;
  const int step = kClipCells * ((nblk - seg + kSeg - 1) / kSeg);   // the segment's blocks
  for (int e = (blk / kSeg) * kClipCells + group; e < queued; e += step) {
    const int i = a.queue[(size_t)seg * a.qcap + e];
    if (i < 0 || i >= a.n || (a.deg[i] != kDegClip && a.deg[i] != kDegNear)) continue;
    clip_cell<WALLS, TIERED>(a, i, s_slots[group]);
    wave_sync();   // the slots are taken by the next cell
  }
}

// ---------------------------------------------------------------------------
// the cell of one point when it keeps its previous neighbours
// ---------------------------------------------------------------------------
// Under the small moves of a time step most cells keep their neighbours, and
// the previous mesh lists them counter-clockwise.  Then the cell's vertices
// are the points equidistant from r_i and two consecutive neighbours, and
// the cell is proved by checking each vertex against every other candidate
// (one dot product), instead of cutting every bisector by every other one.
// The proof holds in exact arithmetic when every consecutive pair turns
// counter-clockwise by less than half a turn (and more than kVertexSin), the
// ring winds once, and every vertex lies inside every other candidate's half
// plane by a margin far above the rounding of the test (kVertexMargin of the
// candidate's half squared distance plus the largest squared vertex distance;
// with one margin for all vertices, the vertex of largest projection on a
// candidate decides for all of them): the polygon is then the intersection of the
// candidates' half planes, and its edges (all of positive length, well above
// the input stage's cut for dropping one) are the ring's neighbours.  The
// candidates are the clip's: the mirrors of a walled box, the ring, and the
// neighbours' neighbours that could reach a vertex.  A cell that fails any
// of these tests (a new neighbour, a lost one, a near-degenerate vertex, a
// ring longer than kGroup or next to a wall) is queued for the clip
// launches (deg = kDegClip), which decide every case.
//
// Of the ring itself only the entries next to a vertex's own two are tried:
// the distance of a convex polygon's vertices from one of its sides grows
// and then falls along the polygon, so those are the nearest ones.
//
// The neighbours' neighbours (about 36 per cell, most of them several times
// over) are most of the loads.  Large meshes therefore try only the ring at
// first (RING), and a second pass (k_rt_near) tries the neighbours'
// neighbours of those cells that have a failed neighbour.  For the others
// they cannot matter where the old mesh is a triangulation (k_rt_near): every
// edge of it at the point or at one of its neighbours is then locally Delaunay, and a point inside a
// vertex's circle would have to be reached from it across such edges only,
// each crossing keeping the point inside the next circle, until a triangle
// holds it as a corner.  (That is a reason, not a proof: the path could leave
// the neighbours' triangles through an edge of two further points.  No mesh
// rests on it: what proves a mesh is its certification, of whichever cells the
// checks left.  Every kept edge is seen by both its cells between the same end
// points (emit and end), so the cells, convex and each about its own point,
// glue to a closed surface over the box that covers it a whole number of times;
// the areas say once, 1e-10 of the box where another sheet would be all of it.
// The cells then tile the box, and |x - r_i|^2 - |x|^2, i the cell of x, is
// continuous and concave across every edge, a bisector, hence concave on the
// box: the least over all points everywhere, which is the Voronoi mesh.)
// The group's loads and stores are contiguous.  (One lane per cell and all candidates at once took
// 1648 us on the 2048 x 2048 wave, bound by the gathers and their address
// arithmetic; the two passes take 367, vector instructions for 260 of them, and
// 205 us over a chain of steps, most of it the gathers of the cells beside a
// failed one: 62 us where none failed.  64 x 64 tube: a chain of 24 dependent
// loads, 38 -> 10 us in one launch.)

// Lane l of a cell's group: ring entry l, its displacement from r_i, and the
// vertex after it.
struct Ring {
  int n, start;       // entries; the entry of least angle
  int c;              // neighbour cell, -1 past the end
  int32_t id;
  double xi, yi, dx, dy, vx, vy;
  double r2;          // largest squared vertex distance of the cell
};

// The ring of cell i (no cell: live = false) and whether it passes every
// test that needs the ring alone.  NB: neighbours from a.nb (an earlier
// launch wrote them), else from the entries' edges; WRITE: written there.
template <bool WALLS, bool NB, bool WRITE>
__device__ __forceinline__ bool load_ring(const Args& a, int i, bool live, Ring& r) {
  const int l = (int)threadIdx.x & (kGroup - 1);
  const double2 pi = a.xy[live ? i : 0];
  r.xi = pi.x;
  r.yi = pi.y;
  int k0 = 0, n = 0;
  if (live) {
    k0 = a.p_off[i];
    const int k1 = a.p_off[i + 1];
    if (k0 >= 0 && k1 >= k0 && k1 <= (NB || WRITE ? a.nb_end : a.p_n_csr)) n = k1 - k0;
  }
  r.c = -1;
  if (l < n) r.c = NB ? a.nb[k0 + l] : prev_neighbour(a, k0 + l);
  if (WRITE) {
    if (l < n) a.nb[k0 + l] = r.c;
    if (n <= kRingMax)   // (a longer row is read by nobody)
      for (int k = l + kGroup; k < n; k += kGroup) a.nb[k0 + k] = prev_neighbour(a, k0 + k);
  }
  if (r.c >= a.n || r.c == i) r.c = -1;   // out of range, or a wall's entry
  const double2 p = a.xy[r.c < 0 ? 0 : r.c];
  r.id = displacement<WALLS>(a, r.xi, r.yi, r.c < 0 ? 0 : r.c, p.x, p.y, r.dx, r.dy);
  bool ok = WALLS ? (r.xi > a.x0 && r.xi < a.x1 && r.yi > a.y0 && r.yi < a.y1)
                  : (r.xi >= a.x0 && r.xi < a.x1 && r.yi >= a.y0 && r.yi < a.y1);
  ok = ok && n >= 3 && n <= kGroup && (l >= n || r.c >= 0);
  r.n = n;

  // vertex l: equidistant from r_i, ring entries l and l+1 (cyclically)
  const int l1 = l + 1 < n ? l + 1 : 0, l2 = l1 + 1 < n ? l1 + 1 : 0, lp = l > 0 ? l - 1 : n - 1;
  const double ax = r.dx, ay = r.dy;
  const double bx = __shfl(ax, l1, kGroup), by = __shfl(ay, l1, kGroup);
  const bool turn = ring_vertex(ax, ay, bx, by, r.vx, r.vy);
  r.r2 = group_max(l < n ? r.vx * r.vx + r.vy * r.vy : 0.0);
  ok = ok && (l >= n || turn);
  // the ring winds once: exactly one step passes angle 0
  const uint32_t wraps = group_bits(l < n && ccw_before(bx, by, ax, ay));
  ok = ok && __popc(wraps) == 1;
  r.start = __ffs(wraps) < n ? __ffs(wraps) : 0;
  // the vertex inside the half planes of the entries beside its own two
  // (the same one for a triangle), by the margin
  const double mr = kVertexMargin * r.r2;
  auto inside = [&](double ux, double uy, double hu) -> bool {
    return hu - (r.vx * ux + r.vy * uy) > kVertexMargin * hu + mr;
  };
  {
    const double ux = __shfl(ax, lp, kGroup), uy = __shfl(ay, lp, kGroup);
    const double wx = __shfl(ax, l2, kGroup), wy = __shfl(ay, l2, kGroup);
    ok = ok && (l >= n || (inside(ux, uy, 0.5 * (ux * ux + uy * uy)) &&
                           inside(wx, wy, 0.5 * (wx * wx + wy * wy))));
  }
  if (WALLS) {
    // the point's mirrors across the walls y0, x1, y1, x0
    const double wy0 = 2.0 * (a.y0 - r.yi), wx1 = 2.0 * (a.x1 - r.xi);
    const double wy2 = 2.0 * (a.y1 - r.yi), wx3 = 2.0 * (a.x0 - r.xi);
    ok = ok && (l >= n || (inside(0.0, wy0, 0.5 * wy0 * wy0) && inside(wx1, 0.0, 0.5 * wx1 * wx1) &&
                           inside(0.0, wy2, 0.5 * wy2 * wy2) && inside(wx3, 0.0, 0.5 * wx3 * wx3)));
  }
  return group_bits(!ok) == 0u;
}

// A cell's vertices and ring ids in LDS, for the lanes of its group (the
// padding keeps the groups of a wave on different banks).
struct Fan {
  double2 v[kGroup + 1];
  int32_t id[kGroup];
};

// Whether every neighbour's neighbour leaves every vertex of a ring that
// passed inside its half plane: one nearer than twice the largest vertex
// distance (with the margin) that is not in the ring is tried.  Lane m goes
// through the entries of ring member m's row.
template <bool WALLS, bool NB>
__device__ __forceinline__ bool second_ring(const Args& a, int i, const Ring& r, Fan& F) {
  const int l = (int)threadIdx.x & (kGroup - 1);
  if (l < r.n) {
    F.v[l] = make_double2(r.vx, r.vy);
    F.id[l] = r.id;
  }
  wave_sync();
  double2 v[kGroup];
  int32_t id[kGroup];
#pragma unroll
  for (int k = 0; k < kGroup; ++k) {   // past the end: the first again
    v[k] = F.v[k < r.n ? k : 0];
    id[k] = F.id[k < r.n ? k : 0];
  }
  const double mr = kVertexMargin * r.r2;
  const double reach = 4.0 * r.r2 * (1.0 + kVertexMargin);
  bool ok = true;
  int l0 = 0, l1 = 0;
  if (r.c >= 0) {
    l0 = a.p_off[r.c];
    l1 = a.p_off[r.c + 1];
    if (l0 < 0 || l1 < l0 || l1 > (NB ? a.nb_end : a.p_n_csr) || l1 - l0 > kRingMax) {
      ok = false;
      l1 = l0;
    }
  }
  constexpr int CH = 8;   // candidates whose loads are in flight together
  for (; l0 < l1; l0 += CH) {
    int c[CH];
    double2 p[CH];
#pragma unroll
    for (int t = 0; t < CH; ++t) c[t] = l0 + t < l1 ? (NB ? a.nb[l0 + t] : a.p_idx[l0 + t]) : -1;
    if (!NB) {
#pragma unroll
      for (int t = 0; t < CH; ++t) c[t] = entry_cell(a, c[t]);
    }
#pragma unroll
    for (int t = 0; t < CH; ++t) {
      if (c[t] >= a.n || c[t] == i) c[t] = -1;
      p[t] = a.xy[c[t] < 0 ? 0 : c[t]];
    }
#pragma unroll
    for (int t = 0; t < CH; ++t) {
      if (c[t] < 0) continue;
      double ux, uy;
      const int32_t u = displacement<WALLS>(a, r.xi, r.yi, c[t], p[t].x, p[t].y, ux, uy);
      const double d2 = ux * ux + uy * uy;
      if (!(d2 < reach)) continue;
      bool known = false;
#pragma unroll
      for (int k = 0; k < kGroup; ++k) known = known || id[k] == u;
      if (known) continue;
      // the largest projection of a vertex on the candidate
      double q = v[0].x * ux + v[0].y * uy;
#pragma unroll
      for (int k = 1; k < kGroup; ++k) q = dmax(q, v[k].x * ux + v[k].y * uy);
      const double hu = 0.5 * d2;
      ok = ok && hu - q > kVertexMargin * hu + mr;
    }
  }
  return group_bits(!ok) == 0u;
}

// Queues the groups' failing cells for the clip, in the queue segment of
// their own block of cells (so that no segment overflows): one atomic per
// wave, whose cells are of one block `home`.
__device__ __forceinline__ void queue_failed(const Args& a, int home, int i, bool failed,
                                             int32_t mark) {
  const int lane = (int)threadIdx.x & 63;
  const bool lead = failed && (lane & (kGroup - 1)) == 0;
  const unsigned long long fails = __ballot(lead);
  if (fails == 0ull) return;
  const int first = __ffsll((long long)fails) - 1;
  const int seg = home % kSeg;
  int base = 0;
  if (lane == first) base = atomicAdd(&a.qcnt[seg * kSegStride], __popcll(fails));
  base = __shfl(base, first);
  if (lead) {
    a.queue[(size_t)seg * a.qcap + base + __popcll(fails & ((1ull << lane) - 1ull))] = i;
    a.deg[i] = mark;
  }
}

// The cells whose ring passes (RING: the ring alone is tried, and the
// neighbours are written for k_rt_near and the clip; else their neighbours
// too).
template <bool B, bool WALLS, bool RING>
__global__ __launch_bounds__(kGroupThreads) void k_rt_vertex(Args one, Batch bt) {
  __shared__ Fan s_fan[RING ? 1 : kThreads];
  int blk;
  const Args& a = block_run<B>(one, bt.cstart, bt, cell_block(), blk);
  if ((a.bc == (int)RICH_BOUNDARY_PERIODIC) == WALLS || tiered(a) != RING)
    return;  // another launch's run
  const int l = (int)threadIdx.x & (kGroup - 1);
  const int i = blk * kThreads + (int)threadIdx.x / kGroup;
  const bool live = i < a.n;
  Ring r;
  bool ok = load_ring<WALLS, false, RING>(a, i, live, r);
  if constexpr (!RING) {
    if (ok) ok = second_ring<WALLS, false>(a, i, r, s_fan[threadIdx.x / kGroup]);
  }
  queue_failed(a, blk, i, live && !ok, kDegClip);
  if (!live || !ok) return;   // whole groups
  // edge l runs from vertex l-1 to vertex l; its slot is its counter-
  // clockwise rank, counted from the entry of least angle
  const int lp = l > 0 ? l - 1 : r.n - 1;
  const double ux = __shfl(r.vx, lp, kGroup), uy = __shfl(r.vy, lp, kGroup);
  const double wx = r.vx, wy = r.vy;
  const double ex = wx - ux, ey = wy - uy;
  const int rank = l >= r.start ? l - r.start : l - r.start + r.n;
  const double cr = l < r.n ? ux * wy - uy * wx : 0.0;
  if (l < r.n) a.s_nb[(size_t)i * kRow + rank] = r.id;
  const double A2 = group_sum(cr);
  const double sx = group_sum(cr * (ux + wx)), sy = group_sum(cr * (uy + wy));
  // (lean_cell of the shortest edge: of every edge, each lane its own)
  const bool lean =
      group_bits(l < r.n && !lean_cell(a, ex * ex + ey * ey, r.r2, 0.5 * A2)) == 0u;
  const uint32_t own = group_bits(l < r.n && i < r.c);
  if (l == 0) {
    a.deg[i] = r.n | (lean ? kLean : 0);
    a.cnt[i] = (uint32_t)r.n | (uint32_t)__popc(own) << 16;   // (if lean)
    a.area[i] = 0.5 * A2;
  }
  if (!lean && l < r.n) {
    double* g = a.s_geo + 3 * ((size_t)i * kMaxFan + rank);
    edge_geometry(r.xi, r.yi, ux, uy, wx, wy, g[0], g[1], g[2]);
  }
  // the cell record, a 16-byte part per lane
  double2* cell = reinterpret_cast<double2*>(a.cells + i);
  if (l == 0) cell[0] = make_double2(r.xi, r.yi);
  const double off = (l == 1 ? sx : sy) / (3.0 * A2);   // (a division for both)
  if (l == 1) cell[1] = make_double2(0.5 * A2, r.xi + off);
  if (l == 2) cell[2] = make_double2(r.yi + off, 0.0);
}

// The neighbours' neighbours of the cells whose ring passed but that have a
// neighbour whose ring did not (or of all, below).  Each wave lists such cells among its own 64
// (a lane per cell), goes through the list kThreads / kGroup cells at a time,
// and queues those that fail for the clip with a mark of their own: the marks
// that others look for stay those of the first pass.
template <bool B, bool WALLS>
__global__ __launch_bounds__(kThreads) void k_rt_near(Args one, Batch bt) {
  constexpr int GROUPS = kThreads / kGroup;
  __shared__ Fan s_fan[GROUPS];
  __shared__ int s_list[kThreads];
  static_assert(kThreads == 64, "a block is one wave");
  int blk;
  const Args& a = block_run<B>(one, bt.cstart, bt, cell_block(), blk);
  if ((a.bc == (int)RICH_BOUNDARY_PERIODIC) == WALLS || !tiered(a))
    return;  // another launch's run
  const int lane = (int)threadIdx.x;
  // Three cells meet at every vertex of the previous mesh just when it has 3 n
  // edges (one more between walls).  Where four meet (an exact lattice, whose
  // diagonal edges of no length were dropped) the rings do not know of the
  // point opposite: every cell is tried.
  const bool whole = a.p_eoff[a.n] == 3 * a.n + (WALLS ? 1 : 0);
  bool near = false;
  const int i0 = blk * kThreads + lane;
  if (i0 < a.n && a.deg[i0] != kDegClip) {
    const int k0 = a.p_off[i0], n = a.p_off[i0 + 1] - k0;   // (3 to kGroup entries, all in range)
    int c[kGroup];
#pragma unroll
    for (int m = 0; m < kGroup; ++m) c[m] = m < n ? a.nb[k0 + m] : i0;
#pragma unroll
    for (int m = 0; m < kGroup; ++m) near = near || !whole || a.deg[c[m]] == kDegClip;
  }
  const unsigned long long nears = __ballot(near);
  if (near) s_list[__popcll(nears & ((1ull << lane) - 1ull))] = i0;
  wave_sync();
  const int count = __popcll(nears), group = lane / kGroup;
  for (int g = group; g - group < count; g += GROUPS) {   // (the whole wave)
    const bool live = g < count;
    const int i = live ? s_list[g] : 0;
    Ring r;
    bool ok = load_ring<WALLS, true, false>(a, i, live, r);
    if (live) ok = second_ring<WALLS, true>(a, i, r, s_fan[group]);
    queue_failed(a, blk, i, live && !ok, kDegNear);
    wave_sync();   // the fans are taken by the next cells
  }
}

// ---------------------------------------------------------------------------
// kept and owned edges of each cell, and their prefix sums.  Offsets are kept
// as a cell's prefix within its scan block (cnt, both counts in one word)
// plus the block's own offset (bsum); emit adds the two and writes off[] and
// eoff[], which spares a launch and a pass over the cells.
// ---------------------------------------------------------------------------
static_assert(kScanThreads * kMaxFan < (1 << 16), "a scan block's counts fit 16 bits");

// Inclusive scan of one value per thread over the block; every thread also
// gets the total.  s holds a value per wave.
template <typename T>
__device__ __forceinline__ T block_scan(T v, T* s, T& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  constexpr int NW = kScanThreads / 64;
  for (int o = 1; o < 64; o <<= 1) {
    const T u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  if (lane == 63) s[wv] = v;
  __syncthreads();
  T before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const T u = s[w];
    if (w < wv) before += u;
    total += u;
  }
  return v + before;
}

// What a block of kScanThreads threads shares while it counts.
struct CountLds {
  uint32_t s[kScanThreads / 64];
  double area[kScanThreads / 64];
  int drop[kScanThreads / 64], walls[kScanThreads / 64];
};

// One thread per cell of scan block blk: the counts (of a lean cell they are
// there already), their scan over the block (into cnt; the total returned to
// every thread) and the block's sums (valid in thread 0).  A slot is kept
// unless its edge is shorter than 1e-12 of the two cells' mean radius; a kept
// edge is owned by its lower cell (by its image code where a cell meets
// itself), a wall's by its cell.
__device__ __forceinline__ uint32_t count_block(const Args& a, int blk, CountLds& S, CPart& c) {
  constexpr int NW = kScanThreads / 64;
  const int i = blk * kScanThreads + threadIdx.x;
  uint32_t v = 0;
  double area = 0.0;
  int drop = 0, walls = 0;
  if (i < a.n) {
    const int di = max(a.deg[i], 0);
    area = a.area[i];
    v = a.cnt[i];
    if (di == 0 || !(area > 0.0)) atomicOr(&a.hdr->flags, RICH_RETESS_CLIP);
    if (!(di & kLean)) {
      const double Ri = sqrt(area / kPi);
      const size_t s0 = (size_t)i * kMaxFan;
      int n_keep = 0, n_own = 0;
      for (int q = 0; q < di; ++q) {
        const int32_t id = slot_nb(a, i, q);
        const int j = (int)((uint32_t)id & kMask);
        const int code = (int)((uint32_t)id >> kShift);
        const bool keep = a.s_geo[3 * (s0 + q)] >= 1e-12 * 0.5 * (Ri + sqrt(a.area[j] / kPi));
        const bool own = code >= kWallX0 || (j != i ? i < j : code >= 5);
        // (a kept slot's rank among the cell's kept ones is its CSR position)
        a.s_flag[s0 + q] = (uint8_t)((keep ? 1 : 0) | (keep && own ? 2 : 0) | (n_keep << 2));
        if (keep) {
          ++n_keep;
          if (own) ++n_own;
          if (code >= kWallX0) ++walls;
        } else {
          ++drop;
        }
      }
      v = (uint32_t)n_keep | (uint32_t)n_own << 16;
    } else {
      walls = (int)(v >> kWallBits);
      v &= (1u << kWallBits) - 1u;
    }
  }
  for (int o = 32; o > 0; o >>= 1) area += __shfl_xor(area, o);
  if (__any(drop != 0 || walls != 0)) {
    for (int o = 32; o > 0; o >>= 1) {
      drop += __shfl_xor(drop, o);
      walls += __shfl_xor(walls, o);
    }
  }
  if ((threadIdx.x & 63) == 0) {
    S.area[threadIdx.x >> 6] = area;
    S.drop[threadIdx.x >> 6] = drop;
    S.walls[threadIdx.x >> 6] = walls;
  }
  uint32_t total;
  const uint32_t inc = block_scan(v, S.s, total);   // (its barrier also publishes the sums)
  if (i < a.n) a.cnt[i] = inc - v;   // (no borrow: both halves grow along the block)
  if (threadIdx.x == 0) {
    c.area = 0.0;
    c.drop = 0;
    c.walls = 0;
    c.pad = 0;
    for (int w = 0; w < NW; ++w) {
      c.area += S.area[w];
      c.drop += S.drop[w];
      c.walls += S.walls[w];
    }
  }
  return total;
}

// The totals into the result header, with the cells queued for the clip and
// the checks that need every cell (areas, capacities); by one thread, kept and
// owned being the totals of both counts, c the sums over all blocks and flags
// the flag word so far.
__device__ __forceinline__ void finish_header(const Args& a, const CPart& c, long long kept,
                                              long long owned, int clipped, int flags) {
  Hdr h = *a.hdr;
  h.flags = flags;
  h.area_sum = c.area;
  h.n_dropped = c.drop;
  h.n_wall = c.walls;
  h.n_csr = kept;
  h.n_edges = owned;
  h.n_clip = clipped;
  if (kept > a.cap_csr || owned > a.cap_edges) h.flags |= RICH_RETESS_CAP;
  if (kept != 2 * owned - c.walls) h.flags |= RICH_RETESS_ASYM;   // an unmatched kept slot
  const double box = a.Lx * a.Ly;
  if (!(fabs(c.area - box) <= 1e-10 * box)) h.flags |= RICH_RETESS_AREA;
  *a.hdr = h;
}
// The cells queued for the clip, in every lane of the calling wave.
__device__ __forceinline__ int queued_cells(const Args& a) {
  int c = 0;
  for (int t = (int)threadIdx.x & 63; t < kSeg; t += 64) c += a.qcnt[t * kSegStride];
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  return c;
}

template <bool B>
__global__ __launch_bounds__(kScanThreads) void k_rt_count(Args one, Batch bt) {
  int blk;
  const Args& a = block_run<B>(one, bt.sstart, bt, blockIdx.x, blk);
  __shared__ CountLds S;
  CPart c;
  const uint32_t total = count_block(a, blk, S, c);
  if (threadIdx.x == 0) {
    a.cpart[blk] = c;
    a.bsum[blk] = total & 0xFFFFu;
    a.bsum[a.n_scan_blocks + blk] = total >> 16;
  }
}

// Small runs (kOneBlockMax scan blocks at most): one block per run counts its
// scan blocks one after another and finishes the header, which spares the
// launch that scans them (16 runs of 900 cells: 4.8 + 5.8 us -> 5.4; four scan
// blocks one after another take 11.6 us against 4.5 + 5.3).  The sums are added
// up as that launch adds them, so that a run's numbers do not depend on which
// way it went.
constexpr int kOneBlockMax = 2;
template <bool B>
__global__ __launch_bounds__(kScanThreads) void k_rt_count_all(Args one, Batch bt) {
  const Args& a = B ? bt.descs[blockIdx.x] : one;
  __shared__ CountLds S;
  __shared__ CPart s_part[kOneBlockMax];
  long long kept = 0, owned = 0;
  const int nb = min(a.n_scan_blocks, kOneBlockMax);
  for (int blk = 0; blk < nb; ++blk) {
    CPart c;
    const uint32_t total = count_block(a, blk, S, c);
    if (threadIdx.x == 0) {
      a.bsum[blk] = kept;
      a.bsum[a.n_scan_blocks + blk] = owned;
      s_part[blk] = c;
    }
    kept += total & 0xFFFFu;
    owned += total >> 16;
    __syncthreads();   // (S is taken by the next block of cells)
  }
  if (threadIdx.x >= 64) return;
  CPart c = {};
  if ((int)threadIdx.x < nb) c = s_part[threadIdx.x];
  for (int o = 32; o > 0; o >>= 1) {
    c.area += __shfl_xor(c.area, o);
    c.drop += __shfl_xor(c.drop, o);
    c.walls += __shfl_xor(c.walls, o);
  }
  const int clipped = queued_cells(a);
  if (threadIdx.x == 0)   // (the flag word as this launch's atomics left it)
    finish_header(a, c, kept, owned, clipped, atomicOr(&a.hdr->flags, 0));
}

// One block: exclusive scan of the block totals, totals, the cells queued for
// the clip counted, and the checks that need every cell (areas, capacities).
// The totals go through one scan over the block's threads (each thread's
// run of scan blocks first); a single thread adding 1024 of them took 22 of
// this kernel's 25 us, the same for every mesh size.
template <bool B>
__global__ __launch_bounds__(kScanThreads) void k_rt_scan_blocks(Args one, Batch bt) {
  const Args& a = B ? bt.descs[blockIdx.x] : one;
  constexpr int NW = kScanThreads / 64;
  __shared__ long long s0[NW], s1[NW];
  __shared__ double s_area[NW];
  __shared__ long long s_drop[NW], s_wall[NW];
  __shared__ int s_clip;
  // the blocks' sums: each thread every kScanThreads-th block, a fixed xor
  // tree over each wave, then thread 0 over the waves in order (a fixed order
  // throughout, so the area sum is reproducible)
  const int nb = a.n_scan_blocks;
  {
    double ar = 0.0;
    long long dr = 0, wl = 0;
    for (int c = threadIdx.x; c < nb; c += kScanThreads) {
      const CPart p = a.cpart[c];
      ar += p.area;
      dr += p.drop;
      wl += p.walls;
    }
    for (int o = 32; o > 0; o >>= 1) {
      ar += __shfl_xor(ar, o);
      dr += __shfl_xor(dr, o);
      wl += __shfl_xor(wl, o);
    }
    if ((threadIdx.x & 63) == 0) {
      s_area[threadIdx.x >> 6] = ar;
      s_drop[threadIdx.x >> 6] = dr;
      s_wall[threadIdx.x >> 6] = wl;
    }
  }
  if (threadIdx.x < 64) {
    const int clipped = queued_cells(a);
    if (threadIdx.x == 0) s_clip = clipped;
  }
  const int per = (nb + kScanThreads - 1) / kScanThreads;
  const int b0 = min(nb, (int)threadIdx.x * per), b1 = min(nb, b0 + per);
  long long c0 = 0, c1 = 0;
  for (int b = b0; b < b1; ++b) {
    c0 += a.bsum[b];
    c1 += a.bsum[nb + b];
  }
  long long t0, t1;
  long long r0 = block_scan(c0, s0, t0) - c0;   // (its barrier also publishes the sums above)
  long long r1 = block_scan(c1, s1, t1) - c1;
  for (int b = b0; b < b1; ++b) {
    const long long u0 = a.bsum[b], u1 = a.bsum[nb + b];
    a.bsum[b] = r0;
    a.bsum[nb + b] = r1;
    r0 += u0;
    r1 += u1;
  }
  if (threadIdx.x == 0) {
    CPart c = {};
    for (int w = 0; w < NW; ++w) {
      c.area += s_area[w];
      c.drop += s_drop[w];
      c.walls += s_wall[w];
    }
    finish_header(a, c, t0, t1, s_clip, a.hdr->flags);
  }
}

// ---------------------------------------------------------------------------
// edge records and CSR entries, certification
// ---------------------------------------------------------------------------
// Length and midpoint of the edge at slot q of cell c (degree word d).
__device__ __forceinline__ void slot_geometry(const Args& a, int c, int d, int q, double& len,
                                              double& mx, double& my) {
  if (!(d & kLean)) {
    const double* g = a.s_geo + 3 * ((size_t)c * kMaxFan + q);
    len = g[0];
    mx = g[1];
    my = g[2];
    return;
  }
  const int n = d & (kLean - 1);
  const double2 pc = a.xy[c];
  double x[3], y[3];   // the slots before, at and after q
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int t = q + k - 1;
    const int32_t id = a.s_nb[(size_t)c * kRow + (t < 0 ? n - 1 : t < n ? t : 0)];
    slot_displacement(a, pc.x, pc.y, id, a.xy[(uint32_t)id & kMask], x[k], y[k]);
  }
  double ux, uy, wx, wy;
  ring_vertex(x[0], y[0], x[1], y[1], ux, uy);
  ring_vertex(x[1], y[1], x[2], y[2], wx, wy);
  edge_geometry(pc.x, pc.y, ux, uy, wx, wy, len, mx, my);
}

// Whether the neighbour at image `to` seen from a cell, its neighbour at
// image `then` and the cell's own neighbour at image `both` are one point (or
// the two cells' mirror images across one wall: the bisector of the cells
// meets the wall in one point).
__device__ __forceinline__ bool same_point(int32_t to, int32_t then, int32_t both) {
  const int c0 = (int)((uint32_t)to >> kShift), c1 = (int)((uint32_t)then >> kShift),
            c2 = (int)((uint32_t)both >> kShift);
  if (c1 >= kWallX0 || c2 >= kWallX0) return c1 == c2;
  if (((uint32_t)(then ^ both) & kMask) != 0u) return false;
  if ((c0 | c1 | c2) == 0) return true;
  int s[3][2] = {};
  if (c0) code_shift(c0, s[0][0], s[0][1]);
  if (c1) code_shift(c1, s[1][0], s[1][1]);
  if (c2) code_shift(c2, s[2][0], s[2][1]);
  return s[0][0] + s[1][0] == s[2][0] && s[0][1] + s[1][1] == s[2][1];
}

// First CSR entry / first owned edge of cell c: its scan block's offset plus
// its own within the block.
__device__ __forceinline__ int csr_offset(const Args& a, int c) {
  return (int)a.bsum[c / kScanThreads] + (int)(a.cnt[c] & 0xFFFFu);
}
__device__ __forceinline__ int edge_offset(const Args& a, int c) {
  return (int)a.bsum[a.n_scan_blocks + c / kScanThreads] + (int)(a.cnt[c] >> 16);
}

// What an edge's owner needs of the neighbour, loaded together: its degree
// word, its row and its first CSR entry.
struct Other {
  int d;
  int32_t id[kRow];
  int k;
};
__device__ __forceinline__ Other load_other(const Args& a, int j) {
  Other o;
  o.d = max(a.deg[j], 0);
  const int4* row = reinterpret_cast<const int4*>(a.s_nb + (size_t)j * kRow);
  const int4 v0 = row[0], v1 = row[1];
  const int32_t id[kRow] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
  for (int t = 0; t < kRow; ++t) o.id[t] = id[t];
  o.k = csr_offset(a, j);
  return o;
}
// Its slot that names `want`, or -1 (what its row holds past its edges is
// ignored).
__device__ __forceinline__ int find_slot(const Args& a, int j, const Other& o, int32_t want) {
  const int n = o.d & (kLean - 1);
  int found = -1;
#pragma unroll
  for (int t = kRow - 1; t >= 0; --t) found = t < n && o.id[t] == want ? t : found;
  for (int t = kRow; found < 0 && t < n; ++t)
    if (slot_nb(a, j, t) == want) found = t;
  return found;
}

// Each cell writes, for every edge it owns (its owned slots in slot order
// from eoff[i]): the edge record, its own CSR entry 2 e at the slot's rank
// among its kept slots, and, unless the edge is a wall, the neighbour's entry
// 2 e + 1 at the rank among the neighbour's kept slots of the slot that sees
// the edge.  In a certified mesh every kept slot is the owned or the other
// side of exactly one owned edge (each owned edge is found in one slot of the
// neighbour, and kept = 2 owned - walls), so each CSR entry is written once,
// and each cell's entries run counter-clockwise (slot order).
//
// Both cells must see the same edge.  Between two lean cells that is so when
// the two points beside the other in both rows are the same ones: the edge
// runs between the same two circumcentres then, and what rounding can put
// between two computations of them is below the tolerance (lean_cell).  Any
// other pair is marked for k_rt_end to compare.
//
// A lane per slot; the geometry of lean cells' edges is computed from the
// points here.  (One kernel compared the stored geometry of every pair and
// another read it again for the records: 550 + 415 us on the 2048 x 2048
// wave, this 372, with its loads in two dependent levels.)
template <bool B>
__global__ __launch_bounds__(kGroupThreads) void k_rt_emit(Args one, Batch bt) {
  int blk;
  const Args& a = block_run<B>(one, bt.cstart, bt, cell_block(), blk);
  const int l = (int)threadIdx.x % kGroup;
  const int i = blk * kThreads + (int)threadIdx.x / kGroup;
  if (i >= a.n) return;  // whole groups
  // the cell's own loads go out together (a row holds kRow slots, read or not)
  const int di = max(a.deg[i], 0);
  static_assert(kGroup == kRow, "a lane per slot of a row");
  const int32_t id0 = a.s_nb[(size_t)i * kRow + l];
  const double2 pi = a.xy[i];
  const int k = csr_offset(a, i);
  int e = edge_offset(a, i);
  const bool failed = a.hdr->flags != 0;   // (offsets may be past the buffers)
  const int d = di & (kLean - 1);
  if (l == 0) {
    a.off[i] = k;
    a.eoff[i] = e;
    if (i == a.n - 1) {   // the totals close the offsets
      a.off[a.n] = (int32_t)a.hdr->n_csr;
      a.eoff[a.n] = (int32_t)a.hdr->n_edges;
    }
  }
  // slot q's match in the neighbour and, if it has one, edge ee: the record
  // and both cells' CSR entries
  bool bad = false, later = false;
  auto put = [&](int q, int rank, int ee, int32_t id, const Other& o, int32_t prev, int32_t next,
                 double len, double mx, double my) {
    const int code = (int)((uint32_t)id >> kShift);
    const int j = (int)((uint32_t)id & kMask);
    int entry = -1;   // of the neighbour
    if (code < kWallX0) {
      const int t = find_slot(a, j, o, pack(i, back_code(code)));
      if (t < 0) {
        bad = true;
        return;
      }
      int place = t;
      later = true;
      if (o.d & kLean) {
        if (di & kLean) {
          const int nj = o.d & (kLean - 1);
          const int tb = t > 0 ? t - 1 : nj - 1, ta = t + 1 < nj ? t + 1 : 0;
          int32_t before = o.id[0], after = o.id[0];
#pragma unroll
          for (int m = 1; m < kRow; ++m) {
            before = m == tb ? o.id[m] : before;
            after = m == ta ? o.id[m] : after;
          }
          later = !(same_point(id, before, next) && same_point(id, after, prev));
        }
      } else {
        const uint8_t f = a.s_flag[(size_t)j * kMaxFan + t];
        if (!(f & 1)) {   // the neighbour drops it
          bad = true;
          return;
        }
        place = f >> 2;
      }
      entry = o.k + place;
    }
    if (failed) return;
    rich_edge r;
    r.fx = mx;
    r.fy = my;
    r.len = len;
    r.i = i;
    r.j = id;
    a.edges[ee] = r;
    a.idx[k + rank] = 2 * ee;
    if (entry >= 0) a.idx[entry] = 2 * ee + 1;
  };
  const uint32_t below = (1u << l) - 1u;
  uint32_t chk = 0;
  if (di & kLean) {   // every slot kept; no image of the cell itself
    const int32_t id = l < d ? id0 : 0;
    const int j = (int)((uint32_t)id & kMask);
    const bool own = l < d && (i < j || (int)((uint32_t)id >> kShift) >= kWallX0);
    const double2 pj = a.xy[j];
    Other o;
    if (own) o = load_other(a, j);
    double dx, dy;
    slot_displacement(a, pi.x, pi.y, id, pj, dx, dy);
    const int ln = l + 1 < d ? l + 1 : 0, lp = l > 0 ? l - 1 : d - 1;
    const int32_t next = __shfl(id, ln, kGroup), prev = __shfl(id, lp, kGroup);
    const double bx = __shfl(dx, ln, kGroup), by = __shfl(dy, ln, kGroup);
    double wx, wy;
    ring_vertex(dx, dy, bx, by, wx, wy);
    const double ux = __shfl(wx, lp, kGroup), uy = __shfl(wy, lp, kGroup);
    const uint32_t mo = group_bits(own);
    if (own) {
      double len, mx, my;
      edge_geometry(pi.x, pi.y, ux, uy, wx, wy, len, mx, my);
      put(l, l, e + __popc(mo & below), id, o, prev, next, len, mx, my);
    }
    chk = group_bits(later);
  } else {
    const size_t s0 = (size_t)i * kMaxFan;
    for (int base = 0; base < d; base += kGroup) {
      const int q = base + l;
      const uint8_t f = q < d ? a.s_flag[s0 + q] : (uint8_t)0;
      const bool own = (f & 3) == 3;
      const uint32_t mo = group_bits(own);
      later = false;
      if (own) {
        const double* g = a.s_geo + 3 * (s0 + q);
        const int32_t id = slot_nb(a, i, q);
        const Other o = load_other(a, (int)((uint32_t)id & kMask));
        put(q, f >> 2, e + __popc(mo & below), id, o, 0, 0, g[0], g[1], g[2]);
      }
      chk |= group_bits(later) << base;
      e += __popc(mo);
    }
  }
  if (l == 0) a.chk[i] = chk;
  if (bad) atomicOr(&a.hdr->flags, RICH_RETESS_ASYM);
}

// Compares the edges that emit left (a thread per cell), and closes the
// rebuild: the last block to finish folds the flags into the sticky word,
// and leaves a failed re-tessellation without edges.  A block's verdict and
// its count go to one word, verdict first, so that the block that completes
// the count holds every verdict without a fence (a device fence writes back
// the L2: 960 us with one in each wave of the 2048 x 2048 wave, 12 without).
constexpr uint32_t kUnlike = 1u << 31;
constexpr int kEndMaxBlocks = 256;   // of one run: the counts meet on one address, 12 ns each
static_assert(kMask / kScanThreads < kUnlike, "the count of a run's blocks stays below the verdict");
template <bool B>
__global__ __launch_bounds__(kScanThreads) void k_rt_end(Args one, Batch bt) {
  int blk;
  const int run = B ? run_of_block(bt.sstart, bt.n_runs, blockIdx.x) : 0;
  const Args& a = block_run<B>(one, bt.sstart, bt, blockIdx.x, blk);
  const int blocks = B ? min(a.n_scan_blocks, kEndMaxBlocks) : gridDim.x;   // of this run
  if (blk >= blocks) return;   // (the whole block)
  __shared__ int s_bad, s_flags;   // s_flags: of a finished rebuild, else 0
  if (threadIdx.x == 0) s_bad = s_flags = 0;
  __syncthreads();
  for (int i = blk * kScanThreads + threadIdx.x; i < a.n; i += blocks * kScanThreads)
  for (uint32_t chk = a.chk[i]; chk != 0u; chk &= chk - 1u) {
    const int q = __ffs(chk) - 1;
    const int32_t id = slot_nb(a, i, q);
    const int j = (int)((uint32_t)id & kMask), code = (int)((uint32_t)id >> kShift);
    const int di = a.deg[i], dj = a.deg[j];
    const int t = find_slot(a, j, load_other(a, j), pack(i, back_code(code)));   // (emit found it)
    if (t < 0) {
      s_bad = 1;
      continue;
    }
    double L, fx, fy, Lj, fxj, fyj;
    slot_geometry(a, i, di, q, L, fx, fy);
    slot_geometry(a, j, dj, t, Lj, fxj, fyj);
    if (code != 0) {  // the neighbour sees the edge one image away
      int sx, sy;
      code_shift(code, sx, sy);
      fxj += sx * a.Lx;
      fyj += sy * a.Ly;
    }
    const double Ri = sqrt(a.area[i] / kPi), Rj = sqrt(a.area[j] / kPi);
    const double tol = 1e-9 * (Ri + Rj);
    if (!(Lj >= 1e-12 * 0.5 * (Ri + Rj)) || fabs(L - Lj) > tol ||
        fabs(fx - fxj) > tol || fabs(fy - fyj) > tol)
      s_bad = 1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_bad) atomicOr(&a.hdr->done, kUnlike);
    const uint32_t w = atomicAdd(&a.hdr->done, 1u);
    if ((w & ~kUnlike) == (uint32_t)blocks - 1u) {
      Hdr h = *a.hdr;   // (nobody else writes the rest of it in this launch)
      if (w & kUnlike) h.flags |= RICH_RETESS_ASYM;
      h.sticky |= h.flags;
      a.hdr->flags = h.flags;
      a.hdr->sticky = h.sticky;
      s_flags = h.flags;
      if (a.flag_out != nullptr) {
        *a.flag_out = h.flags;
        a.info_out->n_edges = h.n_edges;
        a.info_out->n_csr = h.n_csr;
      }
      if (B) {
        bt.hdr_out[run] = h;
        bt.flags_out[run] = h.flags;
      }
    }
  }
  __syncthreads();
  if (s_flags != 0) {
    for (int c = threadIdx.x; c <= a.n; c += kScanThreads) {
      a.off[c] = 0;
      a.eoff[c] = 0;
    }
  }
}

}  // namespace retess

// ===========================================================================
// Host side
// ===========================================================================
// (rich_kernels.hip) two host blocks to device memory through a pinned
// staging ring, enqueued on the stream
namespace rich_host {
int upload2(void* d0, const void* h0, size_t n0, void* d1, const void* h1, size_t n1,
            hipStream_t st);
}
namespace {

size_t rt_align(size_t v) { return (v + 255) / 256 * 256; }

void rt_capacity(int64_t n, int64_t* ce, int64_t* cc) {
  const int64_t r = (int64_t)std::ceil(std::sqrt((double)n));
  *ce = 3 * n + 8 * r + 64;
  *cc = 2 * *ce;
}

struct RtLayout {
  size_t deg, area, s_nb, s_nbx, s_geo, s_flag, cnt, chk, bsum, cpart, qcnt, queue, xy, nbr, total;
  int64_t nbr_cap;
  int nb, qcap;
};

RtLayout rt_layout(int64_t n) {
  RtLayout L;
  const size_t slots = (size_t)n * retess::kMaxFan;
  L.nb = (int)((n + retess::kScanThreads - 1) / retess::kScanThreads);
  size_t o = 256;  // result header
  L.deg = o;    o += rt_align(4 * (size_t)n);
  const size_t row = (size_t)n * retess::kRow, rest = slots - row;
  L.area = o;   o += rt_align(8 * (size_t)n);
  L.s_nb = o;   o += rt_align(4 * row);
  L.s_nbx = o;  o += rt_align(4 * rest);
  L.s_geo = o;  o += rt_align(24 * slots);
  L.s_flag = o; o += rt_align(slots);
  L.cnt = o;    o += rt_align(4 * (size_t)n);
  L.chk = o;    o += rt_align(4 * (size_t)n);
  L.bsum = o;   o += rt_align(16 * (size_t)L.nb);
  L.cpart = o;  o += rt_align(sizeof(retess::CPart) * (size_t)L.nb);
  const int64_t blocks = (n + retess::kThreads - 1) / retess::kThreads;
  L.qcnt = o;   o += rt_align(4 * (size_t)retess::kSeg * retess::kSegStride);
  L.qcap = (int)(retess::kThreads * ((blocks + retess::kSeg - 1) / retess::kSeg));
  L.queue = o;  o += rt_align(4 * (size_t)retess::kSeg * (size_t)L.qcap);
  L.xy = o;     o += rt_align(16 * (size_t)n);
  int64_t ce;
  rt_capacity(n, &ce, &L.nbr_cap);
  L.nbr = o;    o += rt_align(4 * (size_t)L.nbr_cap);
  L.total = o;
  return L;
}

// Whether a rebuild takes this previous mesh at all: its counts, arrays and box
// (periodic: at least 16 cells).
bool takes_mesh(const rich_mesh* m) {
  if (!m || m->n_cells <= 0 || m->n_cells > (int64_t)retess::kMask) return false;
  if (!m->off || !m->eoff || (m->n_csr > 0 && !m->idx) || (m->n_edges > 0 && !m->edges) ||
      m->n_csr < 0 || m->n_edges < 0 || m->n_csr >= (int64_t)INT32_MAX ||
      m->n_edges >= (int64_t)INT32_MAX)
    return false;
  if (!(m->box[2] > m->box[0]) || !(m->box[3] > m->box[1]) || !std::isfinite(m->box[0]) ||
      !std::isfinite(m->box[1]) || !std::isfinite(m->box[2]) || !std::isfinite(m->box[3]))
    return false;
  return m->bc == RICH_BOUNDARY_WALLS || (m->bc == RICH_BOUNDARY_PERIODIC && m->n_cells >= 16);
}

// Checks one run's arguments and fills its descriptor; RICH_OK or the status.
int make_args(const rich_mesh* prev, const double* x, const double* y,
              const rich_mesh_bufs* out, void* ws, size_t ws_bytes, retess::Args& a,
              RtLayout& L) {
  if (!x || !y || !out || !ws || !takes_mesh(prev)) return RICH_E_INVAL;
  const int64_t n = prev->n_cells;
  if (out->n_cells != n) return RICH_E_INVAL;
  if (!out->cells || !out->edges || !out->off || !out->idx || !out->eoff ||
      (reinterpret_cast<uintptr_t>(out->cells) & 15) ||
      (reinterpret_cast<uintptr_t>(out->edges) & 15) || out->cap_edges <= 0 ||
      out->cap_csr <= 0 || out->cap_csr >= (int64_t)INT32_MAX)
    return RICH_E_INVAL;
  L = rt_layout(n);
  if (ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255)) return RICH_E_NOMEM;

  char* w = static_cast<char*>(ws);
  std::memset(&a, 0, sizeof(a));
  a.p_off = prev->off;
  a.p_eoff = prev->eoff;
  a.p_idx = prev->idx;
  a.p_edges = prev->edges;
  a.p_n_csr = prev->n_csr;
  a.p_n_edges = prev->n_edges;
  a.x = x;
  a.y = y;
  a.cells = out->cells;
  a.edges = out->edges;
  a.off = out->off;
  a.idx = out->idx;
  a.eoff = out->eoff;
  a.cap_edges = out->cap_edges;
  a.cap_csr = out->cap_csr;
  a.hdr = reinterpret_cast<retess::Hdr*>(w);
  a.deg = reinterpret_cast<int32_t*>(w + L.deg);
  a.s_nb = reinterpret_cast<int32_t*>(w + L.s_nb);
  a.s_geo = reinterpret_cast<double*>(w + L.s_geo);
  a.s_flag = reinterpret_cast<uint8_t*>(w + L.s_flag);
  a.area = reinterpret_cast<double*>(w + L.area);
  a.s_nbx = reinterpret_cast<int32_t*>(w + L.s_nbx);
  a.chk = reinterpret_cast<uint32_t*>(w + L.chk);
  a.cnt = reinterpret_cast<uint32_t*>(w + L.cnt);
  a.bsum = reinterpret_cast<int64_t*>(w + L.bsum);
  a.cpart = reinterpret_cast<retess::CPart*>(w + L.cpart);
  a.qcnt = reinterpret_cast<int32_t*>(w + L.qcnt);
  a.queue = reinterpret_cast<int32_t*>(w + L.queue);
  a.qcap = L.qcap;
  a.xy = reinterpret_cast<double2*>(w + L.xy);
  a.nb = reinterpret_cast<int32_t*>(w + L.nbr);
  a.nb_cap = L.nbr_cap;
  a.nb_end = std::min(prev->n_csr, L.nbr_cap);
  a.form = n < retess::kTieredMin        ? retess::kOneLaunch
           : prev->n_csr <= L.nbr_cap    ? retess::kTiered
                                         : retess::kByUse;
  a.x0 = prev->box[0];
  a.y0 = prev->box[1];
  a.x1 = prev->box[2];
  a.y1 = prev->box[3];
  a.Lx = a.x1 - a.x0;
  a.Ly = a.y1 - a.y0;
  a.size = std::max(a.Lx, a.Ly);
  for (int k = 0; k < 4; ++k) a.size = std::max(a.size, std::fabs(prev->box[k]));
  a.n = (int32_t)n;
  a.bc = (int32_t)prev->bc;
  a.n_scan_blocks = L.nb;
  return RICH_OK;
}

// The kinds of run a call holds: between walls or periodic, in the one launch
// or the two (a run that the kernels decide on counts as both).
struct Kinds {
  bool has[2][2] = {};   // [walls][two launches]
  void add(const retess::Args& a) {
    bool* h = has[a.bc == (int)RICH_BOUNDARY_PERIODIC ? 0 : 1];
    if (a.form != retess::kTiered) h[0] = true;
    if (a.form != retess::kOneLaunch) h[1] = true;
  }
};

// The launches that find the cells, for one kind of box.
template <bool B, bool WALLS>
void launch_cells(const retess::Args& a, const retess::Batch& bt, int gc, int gq, const bool* forms,
                  hipStream_t st) {
  using namespace retess;
  if (forms[1]) {
    hipLaunchKernelGGL((k_rt_vertex<B, WALLS, true>), dim3(gc), dim3(kGroupThreads), 0, st, a, bt);
    hipLaunchKernelGGL((k_rt_near<B, WALLS>), dim3(gc), dim3(kThreads), 0, st, a, bt);
    hipLaunchKernelGGL((k_rt_clip<B, WALLS, true>), dim3(gq), dim3(kClipThreads), 0, st, a, bt);
  }
  if (forms[0]) {
    hipLaunchKernelGGL((k_rt_vertex<B, WALLS, false>), dim3(gc), dim3(kGroupThreads), 0, st, a, bt);
    hipLaunchKernelGGL((k_rt_clip<B, WALLS, false>), dim3(gq), dim3(kClipThreads), 0, st, a, bt);
  }
}

// The launches of one re-tessellation (B: of n_runs runs at once, with gc cell
// blocks and gs scan blocks in all).
template <bool B>
void launch_all(const retess::Args& a, const retess::Batch& bt, int gc, int gs, int n_runs,
                const Kinds& kinds, bool one_block, hipStream_t st) {
  using namespace retess;
  const int gq = B ? gc : std::min(gc, kClipMaxBlocks);   // (a batch's blocks find their run by gc)
  hipLaunchKernelGGL(k_rt_begin<B>, dim3(gc), dim3(kThreads), 0, st, a, bt);
  launch_cells<B, true>(a, bt, gc, gq, kinds.has[1], st);
  launch_cells<B, false>(a, bt, gc, gq, kinds.has[0], st);
  if (one_block) {
    hipLaunchKernelGGL(k_rt_count_all<B>, dim3(n_runs), dim3(kScanThreads), 0, st, a, bt);
  } else {
    hipLaunchKernelGGL(k_rt_count<B>, dim3(gs), dim3(kScanThreads), 0, st, a, bt);
    hipLaunchKernelGGL(k_rt_scan_blocks<B>, dim3(n_runs), dim3(kScanThreads), 0, st, a, bt);
  }
  hipLaunchKernelGGL(k_rt_emit<B>, dim3(gc), dim3(kGroupThreads), 0, st, a, bt);
  hipLaunchKernelGGL(k_rt_end<B>, dim3(B ? gs : std::min(gs, kEndMaxBlocks)), dim3(kScanThreads),
                     0, st, a, bt);
}

// Batch workspace: descriptors, the two start tables, result headers, flags.
size_t batch_hdr_offset(int32_t n) {
  return rt_align(sizeof(retess::Args) * (size_t)n) + rt_align(8 * ((size_t)n + 1));
}
size_t batch_flags_offset(int32_t n) {
  return batch_hdr_offset(n) + rt_align(sizeof(retess::Hdr) * (size_t)n);
}
size_t batch_bytes(int32_t n) { return batch_flags_offset(n) + rt_align(4 * (size_t)n); }

}  // namespace

namespace {

// rich_retess, its flags and counts also to flag_out and info_out (device; or null)
int retess_one(const rich_mesh* prev, const double* x, const double* y,
               const rich_mesh_bufs* out, void* ws, size_t ws_bytes, int32_t* flag_out,
               rich_retess_info* info_out, hipStream_t st) {
  retess::Args a;
  RtLayout L;
  const int rc = make_args(prev, x, y, out, ws, ws_bytes, a, L);
  if (rc) return rc;
  a.flag_out = flag_out;
  a.info_out = info_out;
  const int64_t n = prev->n_cells;
  const int gc = (int)((n + retess::kThreads - 1) / retess::kThreads);
  Kinds kinds;
  kinds.add(a);
  launch_all<false>(a, retess::Batch{}, gc, L.nb, 1, kinds, L.nb <= retess::kOneBlockMax, st);
  return hipGetLastError() == hipSuccess ? RICH_OK : RICH_E_DEVICE;
}

// rich_retess_batch, likewise (flag_out, info_out: per run, or null)
int retess_many(int32_t n, const rich_mesh* const* prev, const double* const* x,
                const double* const* y, const rich_mesh_bufs* const* out, void* const* ws,
                const size_t* ws_bytes, int32_t* const* flag_out,
                rich_retess_info* const* info_out, void* bws, size_t bws_bytes, hipStream_t st) {
  if (n <= 0 || !prev || !x || !y || !out || !ws || !ws_bytes || !bws) return RICH_E_INVAL;
  if (bws_bytes < batch_bytes(n) || (reinterpret_cast<uintptr_t>(bws) & 255)) return RICH_E_NOMEM;
  std::vector<retess::Args> args((size_t)n);
  std::vector<int32_t> starts(2 * ((size_t)n + 1));
  int64_t gc = 0, gs = 0;
  for (int32_t r = 0; r < n; ++r) {
    RtLayout L;
    const int rc = make_args(prev[r], x[r], y[r], out[r], ws[r], ws_bytes[r], args[r], L);
    if (rc) return rc;
    if (flag_out) {
      args[r].flag_out = flag_out[r];
      args[r].info_out = info_out[r];
    }
    for (int32_t q = 0; q < r; ++q)
      if (ws[q] == ws[r]) return RICH_E_INVAL;   // runs need workspaces of their own
    starts[r] = (int32_t)gc;
    starts[n + 1 + r] = (int32_t)gs;
    gc += (prev[r]->n_cells + retess::kThreads - 1) / retess::kThreads;
    gs += L.nb;
    if (gc >= INT32_MAX / 2 || gs >= INT32_MAX / 2) return RICH_E_INVAL;
  }
  starts[n] = (int32_t)gc;
  starts[2 * (size_t)n + 1] = (int32_t)gs;
  char* b = static_cast<char*>(bws);
  const size_t o_start = rt_align(sizeof(retess::Args) * (size_t)n);
  // the host arrays die with this call: they go through the pinned staging
  // ring, whose copies are enqueued on the stream (no wait)
  const int up = rich_host::upload2(b, args.data(), sizeof(retess::Args) * (size_t)n,
                                    b + o_start, starts.data(), starts.size() * sizeof(int32_t),
                                    st);
  if (up != RICH_OK) return up;
  retess::Batch bt;
  bt.descs = reinterpret_cast<const retess::Args*>(b);
  bt.cstart = reinterpret_cast<const int32_t*>(b + o_start);
  bt.sstart = bt.cstart + n + 1;
  bt.hdr_out = reinterpret_cast<retess::Hdr*>(b + batch_hdr_offset(n));
  bt.flags_out = reinterpret_cast<int32_t*>(b + batch_flags_offset(n));
  bt.n_runs = n;
  bool one_block = true;   // (every run of the batch small)
  Kinds kinds;
  for (const retess::Args& r : args) {
    one_block = one_block && r.n_scan_blocks <= retess::kOneBlockMax;
    kinds.add(r);
  }
  launch_all<true>(args[0], bt, (int)gc, (int)gs, n, kinds, one_block, st);
  return hipGetLastError() == hipSuccess ? RICH_OK : RICH_E_DEVICE;
}

}  // namespace

namespace rich_host {
bool retess_takes(const rich_mesh* prev) { return takes_mesh(prev); }
int retess_reported(const rich_mesh* prev, const double* x, const double* y,
                    const rich_mesh_bufs* out, void* ws, size_t ws_bytes, int32_t* flags,
                    rich_retess_info* info, hipStream_t st) {
  return retess_one(prev, x, y, out, ws, ws_bytes, flags, info, st);
}
int retess_batch_reported(int32_t n, const rich_mesh* const* prev, const double* const* x,
                          const double* const* y, const rich_mesh_bufs* const* out,
                          void* const* ws, const size_t* ws_bytes, int32_t* const* flags,
                          rich_retess_info* const* info, void* bws, size_t bws_bytes,
                          hipStream_t st) {
  return retess_many(n, prev, x, y, out, ws, ws_bytes, flags, info, bws, bws_bytes, st);
}
}  // namespace rich_host

extern "C" {

int rich_retess_capacity(int64_t n_cells, int64_t* cap_edges, int64_t* cap_csr) {
  if (n_cells <= 0 || n_cells > (int64_t)retess::kMask || !cap_edges || !cap_csr)
    return RICH_E_INVAL;
  rt_capacity(n_cells, cap_edges, cap_csr);
  if (*cap_csr >= (int64_t)INT32_MAX) return RICH_E_INVAL;
  return RICH_OK;
}

int rich_retess_workspace_size(int64_t n_cells, size_t* bytes) {
  if (n_cells <= 0 || n_cells > (int64_t)retess::kMask || !bytes) return RICH_E_INVAL;
  *bytes = rt_layout(n_cells).total;
  return RICH_OK;
}

int rich_retess(const rich_mesh* prev, const double* x, const double* y,
                const rich_mesh_bufs* out, void* ws, size_t ws_bytes, void* stream) {
  return retess_one(prev, x, y, out, ws, ws_bytes, nullptr, nullptr,
                    static_cast<hipStream_t>(stream));
}

int rich_retess_view(const rich_mesh_bufs* out, const double box[4], uint32_t bc,
                     rich_mesh* m) {
  if (!out || !box || !m || out->n_cells <= 0) return RICH_E_INVAL;
  m->n_cells = out->n_cells;
  m->n_edges = out->cap_edges;
  m->n_csr = out->cap_csr;
  m->cells = out->cells;
  m->edges = out->edges;
  m->off = out->off;
  m->idx = out->idx;
  m->eoff = out->eoff;
  for (int k = 0; k < 4; ++k) m->box[k] = box[k];
  m->bc = bc;
  return RICH_OK;
}

int rich_retess_batch_workspace_size(int32_t n, size_t* bytes) {
  if (n <= 0 || !bytes) return RICH_E_INVAL;
  *bytes = batch_bytes(n);
  return RICH_OK;
}

int rich_retess_batch(int32_t n, const rich_mesh* const* prev, const double* const* x,
                      const double* const* y, const rich_mesh_bufs* const* out,
                      void* const* ws, const size_t* ws_bytes, void* bws, size_t bws_bytes,
                      void* stream) {
  return retess_many(n, prev, x, y, out, ws, ws_bytes, nullptr, nullptr, bws, bws_bytes,
                     static_cast<hipStream_t>(stream));
}

int rich_retess_batch_result(int32_t n, void* bws, void* stream, rich_retess_info* info,
                             int32_t* status) {
  if (n <= 0 || !bws || !info || !status) return RICH_E_INVAL;
  const size_t o_hdr = batch_hdr_offset(n);
  std::vector<retess::Hdr> h((size_t)n);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(h.data(), static_cast<char*>(bws) + o_hdr, sizeof(retess::Hdr) * (size_t)n,
                     hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return RICH_E_DEVICE;
  for (int32_t r = 0; r < n; ++r) {
    info[r].flags = h[r].flags;
    info[r].sticky = h[r].sticky;
    info[r].n_edges = h[r].n_edges;
    info[r].n_csr = h[r].n_csr;
    info[r].n_dropped = h[r].n_dropped;
    info[r].area_sum = h[r].area_sum;
    info[r].n_clipped = h[r].n_clip;
    status[r] = h[r].flags ? RICH_E_MESH : RICH_OK;
  }
  return RICH_OK;
}

int rich_retess_batch_flags_async(int32_t n, void* bws, void* stream, int32_t* host_flags) {
  if (n <= 0 || !bws || !host_flags) return RICH_E_INVAL;
  if (hipMemcpyAsync(host_flags, static_cast<char*>(bws) + batch_flags_offset(n),
                     sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost,
                     static_cast<hipStream_t>(stream)) != hipSuccess)
    return RICH_E_DEVICE;
  return RICH_OK;
}

int rich_retess_result(void* ws, void* stream, rich_retess_info* info) {
  if (!ws || !info) return RICH_E_INVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  retess::Hdr h;
  if (hipMemcpyAsync(&h, ws, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return RICH_E_DEVICE;
  info->flags = h.flags;
  info->sticky = h.sticky;
  info->n_edges = h.n_edges;
  info->n_csr = h.n_csr;
  info->n_dropped = h.n_dropped;
  info->area_sum = h.area_sum;
  info->n_clipped = h.n_clip;
  return h.flags ? RICH_E_MESH : RICH_OK;
}

}  // extern "C"
