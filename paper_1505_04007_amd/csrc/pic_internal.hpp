// Internal declarations of the gfx950 FDTD-PIC library: kernel argument
// blocks and launchers.  Device state is FP32 in normalised units:
//   lengths in cells, time in steps,
//   E in V/m, Ht = eta0 H in V/m, Jt = (dt/eps0) J in V/m,
//   particle u = gamma v / c (dimensionless), positions in cells.
// With S = c dt / dx the field updates read
//   Ht -= S curl E,      E += S curl Ht - Jt_pol - Jt_b,
//   Jt_pol += cbt E - d Jt_pol,  cbt = 2 (wp dt)^2/(2 + g dt), d = 2 g dt/(2 + g dt),
// which is Eq. 6 / Eq. 8 of the paper rescaled (the increment form keeps
// the small damping d exact when rounded to FP32).
//
// Everything that changes from step to step (which H buffer is current,
// steps since the last sort, which particle buffer set is current, the step
// number) lives in a DevState in device memory and is advanced by the
// kernels themselves.  The argument blocks are therefore fixed for the life
// of a simulation, so a sequence of steps can be captured once in a HIP
// graph, and one launch can serve many simulations (an array of argument
// blocks in device memory).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace pic {

constexpr int PBLOCK = 256;  // particle sort kernels
// Push / deposit: one wavefront per workgroup. Wavefronts of one window take
// very different numbers of reduction rounds, and a workgroup's slot on the
// compute unit is freed only when its last wavefront ends, so single-wave
// workgroups keep the units fuller (8 % faster than 256 threads).
constexpr int PUSH_BLOCK = 64;

// Field-kernel tile shapes (cells along x, y of one z plane per workgroup)
// and tile orders the autotuner chooses from.
// Order 0 numbers tiles x, then y, then z (a plane at a time); order 1 x,
// then z, then y (a band of rows marches through all planes, so the next
// plane's values are still in L2 when its tiles run).  The 256 x 1 shapes take
// runs of 256 cells in memory order, across the ends of rows (order 0: of the
// whole grid; order 1: of a band of BAND_ROWS rows of a plane).
constexpr int N_TILE_SHAPES = 16;
constexpr int TILE_FX[N_TILE_SHAPES] = {64, 64, 128, 256, 32, 64, 128, 32, 64, 64, 128, 256, 32, 64, 128, 32};
constexpr int TILE_FY[N_TILE_SHAPES] = {4, 2, 2, 1, 8, 8, 4, 4, 4, 2, 2, 1, 8, 8, 4, 4};
constexpr int TILE_ZO[N_TILE_SHAPES] = {0, 0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 1};
constexpr int TILE_RUNS = 3, TILE_BAND_RUNS = 11;
// Rows of a band: enough that the rows re-read from the next band are few, few
// enough that a band's plane (nx x 16 cells) is still in an XCD's L2 when the
// next plane's run needs it.  H + E launch pair on 512x256x256 cells: 4, 8, 16
// rows 563, 561, 556 us; 240x96x96: 44.8, 44.7, 41.5 us.
constexpr int BAND_ROWS = 16;

// Division of 0 <= n < 2^31 by a fixed d >= 1: n / d = n m >> s with
// s = 31 + ceil(log2 d), m = floor(2^s / d) + 1 < 2^32 (m d = 2^s + e with
// 0 < e <= d, so n m / 2^s exceeds n / d by n e / (d 2^s) < 1 / d).
struct Div {
    unsigned m;
    int s;
};
inline Div make_div(int d)
{
    int l = 0;
    while ((1ll << l) < d) ++l;
    return {(unsigned)(((1ull << (31 + l)) / (unsigned)d) + 1), 31 + l};
}
__device__ __forceinline__ int div(int n, Div d) { return (int)(((unsigned long long)(unsigned)n * d.m) >> d.s); }

// A batched field launch gives each workgroup this many consecutive tiles of
// one member.  One: a workgroup's tiles run one after another (the next
// tile's loads wait for the last one's stores, which may alias them as far
// as the compiler knows), which costs more than the member lookup (work-unit
// table, argument block, device state) it would share.
constexpr int BATCH_TILES = 1;

// The clock of a step.  Every workgroup of its two field updates reads it.  The
// probe launch at the step's end moves it; or (FieldArgs::tick) the field updates
// do by themselves, and no launch is spent on it: the H update reads (parity,
// since_sort), one extra workgroup of it copies them to (e_parity, e_since), the
// E update reads those and its first workgroup writes the next step's (parity,
// since_sort) and step.
struct DevState {
    int parity;      // H[parity] holds H^{n-1/2} at the start of step n
    int since_sort;  // steps since the last cell sort
    int e_parity;    // with tick: the same for the step's E update
    int e_since;
    int pcur;        // particle buffer set in use
    int pad;
    long long step;  // steps taken: E^step is in memory
    float *P[6];     // set pcur's arrays (x, y, z, ux, uy, uz), written with pcur by the sort
};

// CPML data of one axis.  Coefficients are per position along the axis:
// E-type at node i, H-type at i + 1/2; k* hold 1/kappa.  psi arrays cover
// the two absorbing slabs (2*npml planes) of that axis:
//   x: idx = p + 2npml*(j + ny*k)   y: idx = i + nx*(p + 2npml*k)
//   z: idx = i + nx*(j + ny*p),     p = q < npml ? q : q - (n - 2npml).
// psi[a][0] / psi[a][1] belong to the lower / higher numbered updated
// component whose curl differentiates along a (x: y,z   y: x,z   z: x,y):
// psiE[x][0] is the memory of dHz/dx in the Ey update, psiH[z][1] that of
// dEx/dz in the Hy update, and so on.
struct PmlAxis {
    int on;
    int npml;
    const float *bE, *cE, *kE;
    const float *bH, *cH, *kH;
    float *psiE[2];
    float *psiH[2];
};

struct FieldArgs {
    int nx, ny, nz;
    int tile;    // tile shape index (TILE_FX / TILE_FY)
    int gx, gy;  // tiles along x and y (TILE_BAND_RUNS: runs per band and plane, bands)
    Div dx, dy;     // division by nx and ny (the 256 x 1 shapes), else by gx and by gy
    Div dz;         // by nz
    int per[3];
    float S;
    float *E[3];
    float *H[2][3];  // ping-pong: the H update reads H[parity], writes H[parity ^ 1]
    float *Havg[3];  // (H^{n-1/2} + H^{n+1/2})/2 inside the particle box, or null
    PmlAxis pml[3];
    // Drude polarization current on the metal bounding box [lo, hi)
    int mlo[3], mhi[3];
    float *Jp[3];
    const float2 *coef;  // (cbt, d) per box cell
    // when set, the E update also copies E^n and J_pol^{n-1/2} of the metal
    // box here ([6][box cells], E then J_pol): the reverse pass's snapshot
    float *snap;
    // bunch current: read and cleared inside the particle box (+ margin)
    float *Jb[3];
    unsigned long long *Jq[3];  // the fixed-point form instead of Jb, or null
    double qinv;                // V/m per fixed-point unit
    const int *pbox;  // device [6]: lo x,y,z, hi x,y,z (cells, inclusive), or null
    int *nan_flag;
    int tick;         // the field updates move the clock (0: the probe launch does, or nothing)
    DevState *st;
    int turns;        // tiles of an XCD that it takes in turns with the others (xcd_turns)
};

// One-pass field sweep (E update of step n, then H update of step n + 1).
// Every field is one block with its components FIELD_STRIDE apart; the E-side
// state (E, J_pol, the E-side CPML memories) is read from the *in blocks and
// written to the *out blocks, since a workgroup recomputes its neighbours'
// new E at its edges from their old values.
constexpr int FUSED_ROWS = 2;    // y rows per lane
constexpr int FUSED_PLANES = 16;  // z planes per workgroup
struct FusedArgs {
    int nx, ny, nz;
    int per[3];
    float S;
    int N;                       // cells: component stride of E, H, Havg, J_b
    const float *Ein;            // [3][N] E^n
    float *Eout;                 // [3][N] E^{n+1}
    const float *Hin;            // [3][N] H^{n+1/2}
    float *Hout;                 // [3][N] H^{n+3/2}
    float *Havg;                 // [3][N] (H^{n+1/2} + H^{n+3/2}) / 2 in the particle box, or null
    int pon[3], npml[3];
    const float *tab[3];         // per axis [6][n]: bE, cE, kE, bH, cH, kH
    int slab[3];                 // psi cells per component of an axis
    const float *psiEin[3];      // per axis [2][slab]
    float *psiEout[3];
    float *psiH[3];              // updated in place (one owner per H cell)
    int mlo[3], mhi[3];          // metal box [lo, hi)
    int nbox;                    // metal-box cells: component stride of J_pol
    const float *Jpin;           // [3][nbox] J_pol^{n-1/2}
    float *Jpout;                // [3][nbox] J_pol^{n+1/2}
    const float2 *coef;          // (cbt, d) per metal-box cell
    const float *Jb;             // [3][N] bunch current, or null (read only: cleared afterwards)
    const int *pbox;             // device [6] live-cell box of the last sort, or null
    int *nan_flag;
    DevState *st;
    int gy;                      // y blocks of FUSED_ROWS rows
};

struct PartArgs {
    int n;  // particles; their arrays are the device state's P (the current buffer set)
    int nx, ny, nz;
    int per[3];
    const float *E[3];
    const float *B[3];  // (Ht^{n-1/2} + Ht^{n+1/2}) / 2, valid inside the particle box
    float *Jb[3];
    // fixed-point bunch current (deterministic deposit): integer atomics of
    // round(current * qscale) per particle and slot, or null for the FP32
    // atomics into Jb
    unsigned long long *Jq[3];
    float qscale;
    float S;   // c dt / dx
    float ah;  // q dt / (2 m c), per V/m
    float qd;  // -q w / (eps0 dx^2), V/m
    unsigned long long *pushes;  // one counter per wavefront: [ceil(n / 64)]
    DevState *st;
};

struct SortArgs {
    int n;
    int nx, ny, nz;
    int ncell;
    float *P[2][6];
    int *id[2];
    int *key;
    int *rank;
    int *counts;  // [ncell + 1]
    // per key: runs of that key in the array's current order, and where the
    // (last recorded) run starts; a key with one run is contiguous and keeps
    // its order in the scatter
    int *runs;    // [ncell + 1]
    int *first;   // [ncell + 1]
    int *box;     // [6] bounding box of live cells (lo x, y, z, hi x, y, z)
    int *boxpart; // [6 * count workgroups] each count workgroup's box, reduced into box
    int *scan_tmp;  // [scan_tmp_size(ncell + 1)] the scans' tile sums
    DevState *st;
};

struct ProbeArgs {
    int nprobe, nfreq;
    const int *pidx;      // linear Ez index per probe
    const double *omega;  // rad/s
    int large;            // some |omega| dt is 4 or more: below, no phase comes near 2^45
    double *fre, *fim;
    float *series;        // [series_len * nprobe] or null
    long long series_len;
    double dt;
    const float *Ez;
    // optional FP64 record of Ez at the probes for steps g0+1 .. g0+gn
    // (gser[(n - g0 - 1) * nprobe + p]), used by the gradient's objective
    double *gser;
    long long g0, gn;
    DevState *st;
};

// A particle is live when every coordinate is finite and inside [0, n) (cell
// units); a lost particle stores x = -1.  Every kernel indexes the grid from
// a position only after this test, so non-finite values never become indices.
__device__ __forceinline__ bool live_pos(float x, float y, float z, int nx, int ny, int nz)
{
    return x >= 0.f && x < (float)nx && y >= 0.f && y < (float)ny && z >= 0.f && z < (float)nz;
}

// Cells the particle box is widened by: a particle moves less than S cells
// per step, and its gather / deposit stencil reaches two cells past its own.
__device__ __forceinline__ int box_margin(int since_sort, float S)
{
    return 3 + (int)ceilf((float)(since_sort + 1) * S);
}

// Tiles along x and y of a shape, and the workgroups of a field launch.
inline void tile_grid(int nx, int ny, int shape, int &gx, int &gy)
{
    const bool band = shape == TILE_BAND_RUNS;
    gx = band ? (int)(((long long)nx * std::min(BAND_ROWS, ny) + 255) / 256) : (nx + TILE_FX[shape] - 1) / TILE_FX[shape];
    gy = band ? (ny + BAND_ROWS - 1) / BAND_ROWS : (ny + TILE_FY[shape] - 1) / TILE_FY[shape];
}

inline int field_tiles(int nx, int ny, int nz, int shape = 0)
{
    if (shape == TILE_RUNS) return (int)(((long long)nx * ny * nz + 255) / 256);
    int gx, gy;
    tile_grid(nx, ny, shape, gx, gy);
    return gx * gy * nz;
}

// The shape a grid gets before any tuning.  Runs of memory order leave no lane
// idle at the ends of rows and load aligned, and plane by plane the XCDs keep a
// large plane's values between them (xcd_turns).  H + E launch pair, plane runs /
// band runs / 64 x 4 cells: 281x1x3601 cells 17.9 / 24.8 / 25.9 us, 91x45x53 7.9 /
// 8.1 / 9.0, 208x80x80 27.7 / 27.5 / 32.4, 301x203x157 144.7 / 165.8 / 162.9,
// 448x128x128 104.9 / 112.0 / 107.3, 512x256x256 504 / 513 / 519.
constexpr int DEFAULT_TILE = TILE_RUNS;

// How the 8 XCDs share the tiles.  A contiguous block each keeps a block's
// neighbour planes in one L2, but the first and the last then have the absorbing
// slabs of the axis that the order goes through last (and one has the metal film)
// to themselves, and the others wait for them.  So where those slabs fill a quarter
// of such a block or more, the XCDs take turns at chunks of 16 tiles.  They also do
// plane by plane above 2^15 cells a plane, where one plane of 36 bytes a cell no
// longer stays in one L2 but, shared by turns, does in all eight.
// H + E pair and adjoint pair, blocks / turns, order by plane: a batch of 16 of
// 176x64x64 and up 381 / 361 us, 128x64x64 15.3 / 15.2 and 26.0 / 21.8; but 281x1x3601
// with slabs of 10 of 450 planes 19.0 / 20.8, 96x64x96 without slabs 17.2 / 17.8,
// 91x45x53 (848 tiles) 10.0 / 10.2 and 12.4 / 12.6.  (A batch takes turns when they pay
// for a member: 16 of 64x64x64 cells without slabs, a step, 62 / 70 us, of 128x64x64 113
// / 133.)  Large planes, band runs in blocks / plane runs by turns, no slabs: 512x256x256
// 436 / 404, 301x203x157 145.7 / 128.5, 200x200x600 333 / 274, 448x128x128 88.8 / 92.4;
// all slabs: 553 / 504 (bands by turns 513), 172.5 / 144.7, (by turns) 368 / 311, 114.3
// / 104.9.
// Where the line lies, a whole step without slabs, blocks / turns: 128x128x128 28.0 /
// 29.5 us, 160x160x128 41.8 / 41.8, 190x180x64 29.3 / 29.9, 192x192x192 88.4 / 81.9,
// 448x128x128 93.3 / 87.1 (plane runs both), 256x256x16 16.2 / 14.6; few planes:
// 1024x256x6 24.1 / 22.1, 2048x2048x2 115.8 / 103.4, but 2048x2048x1 50.2 / 51.8.
// Band runs by turns of 11, 16, 19, 32, 43, 64 tiles on 512x256x256: 609, 547, 601,
// 598, 589, 572 (16 is half a band's plane there).
constexpr int XCD_CHUNK = 16;
inline int xcd_turns(long long tiles) { return (int)(tiles / (8 * XCD_CHUNK)) * XCD_CHUNK; }
inline bool turns_pay(long long plane, int n, const PmlAxis &slow)
{
    return plane > (1 << 15) || (slow.on && 32LL * slow.npml >= n);
}
inline int xcd_turns(long long tiles, long long plane, int n, const PmlAxis &slow)
{
    return tiles >= 1024 && turns_pay(plane, n, slow) ? xcd_turns(tiles) : 0;
}

// The same for a's grid in the order of its tile shape.
inline bool turns_pay(const FieldArgs &a)
{
    const int slow = TILE_ZO[a.tile] ? 1 : 2;
    return turns_pay(slow == 1 ? 0 : (long long)a.nx * a.ny, slow == 1 ? a.ny : a.nz, a.pml[slow]);
}

// (a's sizes and slabs are set)
inline void set_tile(FieldArgs &a, int shape)
{
    a.tile = shape;
    tile_grid(a.nx, a.ny, shape, a.gx, a.gy);
    const bool runs = shape == TILE_RUNS, band = shape == TILE_BAND_RUNS;
    a.dx = make_div(runs || band ? a.nx : a.gx);
    a.dy = make_div(runs ? a.ny : band ? a.gx : a.gy);
    a.dz = make_div(a.nz);
    const int tiles = field_tiles(a.nx, a.ny, a.nz, shape);
    a.turns = tiles >= 1024 && turns_pay(a) ? xcd_turns(tiles) : 0;
}

// Work units of one member in a batched field launch.
inline long long batch_field_units(int nx, int ny, int nz, int shape)
{
    return ((long long)field_tiles(nx, ny, nz, shape) + BATCH_TILES - 1) / BATCH_TILES;
}

// Quotient and remainder of a small step past a row's (or plane's) start:
// q, r of 0 <= n < d + 256 by d.
__device__ __forceinline__ int step_div(int &n, int d)
{
    int q;
    if (d >= 256) {
        q = n >= d ? 1 : 0;
    } else {
        // n < 511: (n + 1/2) / d is at least 1 / (2 d) off an integer
        q = (int)(((float)n + 0.5f) * (1.f / (float)d));
    }
    n -= q * d;
    return q;
}

// Cell tid of the run of cells starting at c: (i, j, k) in memory order.
__device__ __forceinline__ void run_cell(int c, int tid, int nx, int ny, Div dx, Div dy, int &i, int &j, int &k)
{
    const int r = div(c, dx), k0 = div(r, dy);
    i = c - r * nx + tid;
    j = r - k0 * ny + step_div(i, nx);
    k = k0 + step_div(j, ny);
}

// Linear offset to the neighbour at distance d = +-1 along an axis of n
// cells with stride st: wraps on a periodic axis; across a wall it points
// at the cell itself and clears `ok` (the neighbour value is then 0).
__device__ __forceinline__ int nb_off(int i, int d, int n, int per, int st, bool &ok)
{
    const int r = i + d;
    const bool in = r >= 0 && r < n;
    ok = in || per;
    const int w = r < 0 ? r + n : r - n;
    return in ? d * st : (per ? (w - i) * st : 0);
}

// Global-memory pointers.  A pointer the kernels read from device memory (the
// batched entry points' argument blocks) or pass through a scalar-register
// pin is generic to the compiler, which then emits flat loads, stores and
// atomics: 64-bit vector addresses, and counted with the scalar loads, so a
// wait for either waits for both.  Every pointer the library hands its kernels
// addresses global memory (the same bits), so accesses go through G(p).
template <class T>
using gp = __attribute__((address_space(1))) T *;
template <class T>
__device__ __forceinline__ gp<T> G(T *p)
{
    return (gp<T>)p;
}
// Two floats as a plain vector (HIP's float2 is a class, which C++ cannot
// copy out of a global-typed lvalue).
typedef float fvec2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void gatomic_add(gp<float> p, float v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gatomic_add(gp<unsigned long long> p, unsigned long long v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroup b of B -> tile with XCD locality: the 8 XCDs receive workgroups
// round robin, so workgroup b runs on XCD b % 8; give each XCD a contiguous
// block of tiles.
__device__ __forceinline__ int xcd_block(int b, int B)
{
    const int x = b & 7, q = B >> 3, r = B & 7;
    return x * q + min(x, r) + (b >> 3);
}

// The same with the first `turns` tiles of every XCD in chunks of XCD_CHUNK, the
// XCDs taking turns (xcd_turns).
__device__ __forceinline__ int xcd_tile(int b, int B, int turns)
{
    const int x = b & 7, i = b >> 3;
    if (i < turns) return (i / XCD_CHUNK * 8 + x) * XCD_CHUNK + i % XCD_CHUNK;
    return 8 * turns + xcd_block(b - 8 * turns, B - 8 * turns);
}

// xcd_tile() with each XCD walking its tiles from the end: a launch that
// follows one in the forward order starts on the tiles the other wrote last,
// which are still in the Infinity Cache.
__device__ __forceinline__ int xcd_tile_rev(int turns)
{
    const int B = gridDim.x, x = blockIdx.x & 7, i = blockIdx.x >> 3;
    const int len = (B >> 3) + (x < (B & 7) ? 1 : 0);
    return xcd_tile(8 * (len - 1 - i) + x, B, turns);
}

// Position of plane q inside the two absorbing slabs of an axis.
__device__ __forceinline__ int slab_p(int q, int n, int np) { return q < np ? q : q - (n - 2 * np); }

// launchers (stream-ordered, no synchronisation)
void launch_fused(const FusedArgs &a, hipStream_t s);
void launch_jb_clear(float *Jb, int N, int nx, int ny, int nz, const int *per, const int *pbox, float S,
                     const DevState *st, hipStream_t s);
// The H update.  With a.tick and `probe`, its launch also samples E for the step
// before (extra workgroups, so that the probes cost no launch of their own).
void launch_h_update(const FieldArgs &a, const ProbeArgs *probe, hipStream_t s);
void launch_e_update(const FieldArgs &a, hipStream_t s);
void launch_push_deposit(const PartArgs &a, int mode, hipStream_t s);
// The probes of the step just taken, as a launch of its own; advance: it also
// moves the clock (FieldArgs::tick 0).
void launch_probe(const ProbeArgs &a, bool advance, hipStream_t s);
void launch_fill_i32(int *p, int v, long long n, hipStream_t s);
void launch_sort(const SortArgs &a, int *scan_tmp, hipStream_t s);
// The sorts of nmem simulations (every one with particles) in one launch per
// kernel: args[nmem] on the device, own[nown] the count and scatter
// workgroups (member << 24 | workgroup index in that member).
void launch_sort_batch(const SortArgs *args, const int *own, int nown, int nmem, hipStream_t s);
int scan_tmp_size(long long n);

// Batched forms: one launch over many simulations.  `args` is a device array
// of per-simulation argument blocks; `own` a device table with one entry per
// work unit of the launch (field tile / particle workgroup, `total` of them):
// simulation index << 24 | the unit's index within that simulation.
// turns: the XCDs take turns at the units (xcd_turns), which a batch does when it pays
// for one of its members.
void launch_h_update_batch(const FieldArgs *args, const int *own, int total, int shape, bool turns,
                           const ProbeArgs *probe, int nmem, hipStream_t s);
void launch_e_update_batch(const FieldArgs *args, const int *own, int total, int shape, bool turns, hipStream_t s);
void launch_push_deposit_batch(const PartArgs *args, const int *own, int total, int mode, hipStream_t s);
void launch_probe_batch(const ProbeArgs *args, int n, hipStream_t s);

// ---- reverse-time adjoint of the linear field step (bunch current fixed) ----
//
// Adjoint state in the same normalised units and compact layout as the
// forward fields: Ea = dL/dE, Ha = dL/dHt, Ja = dL/dJt_pol (metal box);
// psiEa / psiHa are the adjoint CPML memories (same slab layout as psiE /
// psiH), DE / DH per-step scratch holding the adjoint weight of each slab
// difference.
struct AdjArgs {
    int nx, ny, nz;
    Div dx, dy;  // division by nx and ny: one thread per cell, in memory order
    int turns;   // as in FieldArgs
    int per[3];
    float S;
    float *Ea[3];
    float *Ha[3];
    PmlAxis pml[3];  // forward coefficient tables (b, c, 1/kappa) and slab sizes
    float *psiEa[3][2], *psiHa[3][2];
    float *DE[3][2], *DH[3][2];
    int mlo[3], mhi[3];
    float *Ja[3];
    const float2 *coef;  // (cbt, d) per metal-box cell
    const float *traj;   // this step's E^n (3 comps) then Jt^{n-1/2} (3 comps), metal box
    double *gcb, *gd;    // per metal-box cell: dL/dcbt and dL/dd summed over its edges
    int nprobe;
    const int *pidx;
    const float *seed;   // dL/dEz at the probes for E^n, or null
    int mode;            // bit 0: reverse the step; bit 1: add seed and prepare the CPML weights
};

// Copy of a box [lo, lo + w) of three grid arrays to / from a packed buffer.
struct BoxCopyArgs {
    float *grid[3];
    float *packed;  // [3][w0*w1*w2], x fastest
    int nx, ny;
    int lo[3], w[3];
    int to_grid;
};

// Forward values the gradient needs at step n on the metal box.
void launch_adj_face(const AdjArgs &a, hipStream_t s);
void launch_adj_edge(const AdjArgs &a, hipStream_t s);
void launch_box_copy(const BoxCopyArgs &a, hipStream_t s);

// FP64 diagnostics
struct DiagArgs {
    int nx, ny, nz;
    int per[3];
    int npml[3];
    int mlo[3], mhi[3];
    const float *E[3];
    const float *H[3];
    int np;
    const float *x, *y, *z, *ux, *uy, *uz;
    double *rho;        // (nx+1)(ny+1)(nz+1) nodes, x fastest
    const double *rho0; // same layout or null
    double qw_over_vol; // q w / dx^3
    double eps0_over_dx;
    double *acc;        // reduction outputs
};
void launch_rho(const DiagArgs &a, hipStream_t s);
void launch_diag_reduce(const DiagArgs &a, hipStream_t s);

// The particle counters of pic_stats: out[2 b], out[2 b + 1] = live particles and
// pushes of workgroup b < the number returned, then the box (6 int) at out + 2
// STATS_BLOCKS.
constexpr int STATS_BLOCK = 1024, STATS_BLOCKS = 256, STATS_WORDS = 2 * STATS_BLOCKS + 3;
int launch_stats(const DiagArgs &a, const unsigned long long *pushes, int nslots, const int *box,
                 unsigned long long *out, hipStream_t s);

// ---- probes ----

// The first 1216 bits of 2 / pi, after 64 zero bits.
static __device__ const unsigned long long TWO_OVER_PI[20] = {
    0ull,
    0xa2f9836e4e441529ull, 0xfc2757d1f534ddc0ull, 0xdb6295993c439041ull, 0xfe5163abdebbc561ull,
    0xb7246e3a424dd2e0ull, 0x06492eea09d1921cull, 0xfe1deb1cb129a73eull, 0xe88235f52ebb4484ull,
    0xe99c7026b45f7e41ull, 0x3991d639835339f4ull, 0x9c845f8bbdf9283bull, 0x1ff897ffde05980full,
    0xef2f118b5a0a6d1full, 0x6d367ecf27cb09b7ull, 0x4f463f669e5fea2dull, 0x7527bac7ebe5f17bull,
    0x3d0739f78a5292eaull, 0x6bfb5fb11f8d5d08ull, 0x56033046fc7b6babull};

// |x| = m 2^e >= 2^45 less the nearest multiple of pi/2, and that multiple mod 4 (M.
// Payne and R. Hanek, Radian reduction for trigonometric functions, 1983): the bits
// of 2/pi above weight 2^(1-e) add multiples of 4 to 2/pi |x|, those more than 192
// bits further down less than 2^-137, so m times the 192 bits between, mod 2^192, has
// the multiple in its top 2 bits and the fraction below.
__device__ __forceinline__ double reduce_large(double x, int &q)
{
    const unsigned long long bits = (unsigned long long)__double_as_longlong(x);
    const int e = (int)((bits >> 52) & 2047) - 1075;
    const unsigned long long m = (bits & ((1ull << 52) - 1)) | (1ull << 52);
    const int b = e + 62, w = min(b >> 6, 16), sh = b & 63;
    unsigned long long v[3];
    for (int k = 0; k < 3; ++k) {
        const unsigned long long hi = TWO_OVER_PI[w + k], lo = TWO_OVER_PI[w + k + 1];
        v[k] = sh ? hi << sh | lo >> (64 - sh) : hi;
    }
    const unsigned long long p0 = m * v[2], c0 = __umul64hi(m, v[2]);
    const unsigned long long p1 = m * v[1] + c0, c1 = __umul64hi(m, v[1]) + (p1 < c0);
    const unsigned long long p2 = m * v[0] + c1;
    const long long hi = (long long)(p2 << 2 | p1 >> 62);
    const unsigned long long lo = p1 << 2 | p0 >> 62;
    const double r = 1.5707963267948965580 * ((double)hi * 0x1p-64 + (double)lo * 0x1p-128);
    const int n = (int)(p2 >> 62) + (hi < 0 ? 1 : 0);
    q = (x < 0.0 ? -n : n) & 3;
    if (!(fabs(x) < INFINITY)) return x - x;
    return x < 0.0 ? -r : r;
}

// |x| < 2^45 less the nearest multiple n of pi/2, and n mod 4: pi/2 as a sum of two
// doubles, each product exact in the fma (n times what they leave out of pi/2 is below
// 4e-20).
__device__ __forceinline__ double reduce_phase(double x, int &q)
{
    const double n = rint(x * 0.63661977236758134308);
    q = (int)(n - 4.0 * floor(0.25 * n));
    return fma(-n, 6.123233995736766036e-17, fma(-n, 1.5707963267948965580, x));
}

// sin and cos of r + q pi/2 by the Taylor series on [-pi/4, pi/4] (the first terms left
// out are below 1e-19).  The library functions would take the field kernel that carries
// the probes to twice its registers.
__device__ __forceinline__ void sincos_reduced(double r, int q, double &sn, double &cs)
{
    const double z = r * r;
    double s = -1.0 / 121645100408832000.0, c = -1.0 / 6402373705728000.0;  // -1/19!, -1/18!
    s = fma(s, z, 1.0 / 355687428096000.0);
    c = fma(c, z, 1.0 / 20922789888000.0);
    s = fma(s, z, -1.0 / 1307674368000.0);
    c = fma(c, z, -1.0 / 87178291200.0);
    s = fma(s, z, 1.0 / 6227020800.0);
    c = fma(c, z, 1.0 / 479001600.0);
    s = fma(s, z, -1.0 / 39916800.0);
    c = fma(c, z, -1.0 / 3628800.0);
    s = fma(s, z, 1.0 / 362880.0);
    c = fma(c, z, 1.0 / 40320.0);
    s = fma(s, z, -1.0 / 5040.0);
    c = fma(c, z, -1.0 / 720.0);
    s = fma(s, z, 1.0 / 120.0);
    c = fma(c, z, 1.0 / 24.0);
    s = fma(s, z, -1.0 / 6.0);
    c = fma(c, z, -0.5);
    s = fma(r * z, s, r);
    c = fma(z, c, 1.0);
    const double a = q & 1 ? c : s, b = q & 1 ? s : c;
    sn = q & 2 ? -a : a;
    cs = q == 1 || q == 2 ? -b : b;
}

// F_p(w_m) += dt Ez_p^n exp(-i w_m n dt) for the newest field E^n, n = n1 steps
// taken (Sec. IV, Figs. 6-7: Ez at the film surface and its spectrum), by one
// workgroup of nt threads; the phase is evaluated directly in FP64 each step.
// LARGE: phases may be 2^45 or more (ProbeArgs::large).
template <int LARGE>
__device__ __forceinline__ void probe_dft(const ProbeArgs &a, long long n1, int t, int nt)
{
    const gp<const float> Ez = G(a.Ez);
    const gp<const int> pidx = G(a.pidx);
    const double tn = (double)n1 * a.dt;
    for (int q = t; q < a.nprobe * a.nfreq; q += nt) {
        const int p = q / a.nfreq, f = q - p * a.nfreq;
        const double ez = (double)Ez[pidx[p]], x = G(a.omega)[f] * tn;
        int k;
        double sn, cs, r = reduce_phase(x, k);
        if (LARGE && !(fabs(x) < 0x1p45)) r = reduce_large(x, k);
        sincos_reduced(r, k, sn, cs);
        G(a.fre)[q] += a.dt * ez * cs;
        G(a.fim)[q] -= a.dt * ez * sn;
    }
    for (int p = t; p < a.nprobe; p += nt) {
        if (a.series && n1 - 1 < a.series_len) G(a.series)[(n1 - 1) * a.nprobe + p] = Ez[pidx[p]];
        if (a.gser && n1 > a.g0 && n1 <= a.g0 + a.gn) G(a.gser)[(n1 - a.g0 - 1) * a.nprobe + p] = (double)Ez[pidx[p]];
    }
}

}  // namespace pic
