// gfx950 kernels of libfwi for grids and batches that do not fill the chip
// with the z sweeps of fwi_kernels.hip: several time steps per launch, the
// wavefields of a tile held in LDS and registers.
//
// Why another form.  The z sweeps give a wavefront 64 columns and walk it
// down 8 + tile rows one after the other; each row costs about 0.4 us of
// latency, so a launch lasts 12 us on a 40 x 32 padded grid and 30 us on a
// 240 x 140 one whatever the work in it.  Here a workgroup owns a tile and
// computes every cell of it at once: a step is one pass over its cells to a
// barrier (two where LDS holds the fields once: two rows of both fields or of
// Born modelling per thread, four rows), and T steps share one launch and one
// read and write of the fields.
//
// Tiling.  A workgroup computes a region of RX x RZ cells.  The tile it owns
// is the region without a margin of 4 T cells on the sides where the grid
// goes on: there the region's edge misses its neighbours, and each step
// carries the error 4 cells further in.  On the grid's own boundary the
// cells outside are zeros, there is no margin, and a grid that fits one
// region runs its whole record in one launch.  The fields are read from one
// set of levels and written to the other, because neighbouring tiles read the
// margins.
//
// A thread holds a patch of PZ rows x 4 columns: the wavefield's rows go
// through LDS as float4 (one 16-byte read serves four cells), the second
// state, w and the accumulators stay in registers over the steps.  Every
// update has the operations of the z sweeps in their order, so both forms
// give the same bits (the damped cells' FP64 division by 1 + g is a product
// with its reciprocal and one correction, which rounds the same).
//
// What bounds it: vector instructions (20 for a cell's Laplacian, 2 moves from
// the neighbouring lanes, the update, in the sponge in FP64; 54 of 64
// lane-operations per clock and CU measured for plain FMAs) times the margin's
// repeated cells, and 6 us (forward) or 8 us (reverse) of launch, load and
// store per T steps.
// Measured per time step, forward / reverse, against the one-step z sweeps
// with their default 16- to 64-row tiles: 1 shot of 240 x 140 cells 2.3 / 3.6
// us (27 / 31), 16 shots of 288 x 128 4.0 / 7.4 us (24 / 30), 4 shots of
// 1088 x 448 11 / 20 us (56 / 61); a 40 x 32 grid 1.2 / 1.6 us (12 / 16).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fwi_internal.h"
#include "fwi_quotient.h"

namespace fwi {
namespace {

__device__ __forceinline__ float bck(int k) {
  return k == 1 ? 8.0f / 5.0f : (k == 2 ? -1.0f / 5.0f : (k == 3 ? 8.0f / 315.0f : -1.0f / 560.0f));
}

// workgroup barrier that orders LDS only: global loads and stores in flight stay
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The value of the lane before / after this one in its row of 16, zero past
// the row's end (every lane of the wavefront must be active).
constexpr int kDppRight1 = 0x111, kDppLeft1 = 0x101;  // row_shr:1, row_shl:1
template <int CTRL>
__device__ __forceinline__ float from_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// blockIdx -> (slot, tile): with a multiple of 8 slots the tiles of a slot
// stay on one XCD (their margins are re-read from its L2)
__device__ __forceinline__ void map_block(const BlockArgs& a, int& slot, int& tile) {
  const int nb = a.nbx * a.nbz, b = blockIdx.x;
  if (a.s.xcd_map) {
    const int r = b >> 3;
    slot = (r / nb) * 8 + (b & 7);
    tile = r % nb;
  } else {
    slot = b / nb;
    tile = b % nb;
  }
}

// A thread's patch and its place in the grid.
template <int RX, int RZ, int PZ>
struct Patch {
  static_assert(RX == 64, "a row of patches is a DPP row of 16 lanes");
  static constexpr int LF = (RZ + 2 * kRadius) * RX;   // LDS floats of one field (4 rows above and below)
  static constexpr int NT = RX / 4 * (RZ / PZ);
  int lx, lz;       // first cell in the region
  int xs, z;        // its storage column and padded row
  int lo;           // its LDS offset
  bool in[PZ];      // rows inside the grid (their columns exist in the storage)
  uint32_t own, model;  // bits 4 i + j: owned / model cells
  int own_x0, own_x1, own_z0, own_z1;  // owned storage columns and padded rows

  __device__ __forceinline__ Patch(const BlockArgs& a, const Dims& d, int tile) {
    const int bx = tile % a.nbx, bz = tile / a.nbx, H = kRadius * a.T;
    const int cs0 = a.c0 + bx * a.sx, rz0 = d.ztop + bz * a.sz;
    own_x0 = bx == 0 ? cs0 : cs0 + H;
    own_x1 = bx == a.nbx - 1 ? d.P : cs0 + a.sx + H;
    own_z0 = bz == 0 ? rz0 : rz0 + H;
    own_z1 = bz == a.nbz - 1 ? d.Z : rz0 + a.sz + H;
    const int t = threadIdx.x;
    lx = 4 * (t % (RX / 4));
    lz = PZ * (t / (RX / 4));
    xs = cs0 + lx;
    z = rz0 + lz;
    lo = (lz + kRadius) * RX + lx;
    own = model = 0;
    const bool xin = xs < d.P;
#pragma unroll
    for (int i = 0; i < PZ; ++i) {
      in[i] = xin && z + i < d.Z;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t bit = 1u << (4 * i + j);
        if (in[i] && z + i >= own_z0 && z + i < own_z1 && xs + j >= own_x0 && xs + j < own_x1) own |= bit;
        if (in[i] && depth_z(d, i) == 0 && depth_x(d, j) == 0) model |= bit;
      }
    }
  }
  // cells into the sponge along z and x
  __device__ __forceinline__ int depth_z(const Dims& d, int i) const {
    return max(max(d.N - (z + i), z + i - (d.N + d.nz - 1)), 0);
  }
  __device__ __forceinline__ int depth_x(const Dims& d, int j) const {
    const int x = xs + j - d.off;
    return max(max(d.N - x, x - (d.N + d.nx - 1)), 0);
  }
  // sponge table entries of a row's cells (columns past the grid, whose w is
  // 0, take the last one)
  template <class T>
  __device__ __forceinline__ void sponge(const Dims& d, const T* tab, int i, T (&t)[4]) const {
    const int dz = depth_z(d, i);
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = tab[min(max(dz, depth_x(d, j)), d.N)];
  }
  // A copy whose indices and masks are computed where they are used: rare or
  // final accesses, whose addresses would otherwise live in registers over
  // the whole loop.
  __device__ __forceinline__ Patch here() const {
    Patch q = *this;
    asm volatile("" : "+v"(q.z), "+v"(q.xs), "+v"(q.own), "+v"(q.model));
    return q;
  }
  // a whole row of the patch is owned or none of it (owned ranges are
  // multiples of 4 columns from the region's first)
  __device__ __forceinline__ bool own_row(int i) const { return (own >> (4 * i)) & 1u; }
  __device__ __forceinline__ bool is_model(int i, int j) const { return (model >> (4 * i + j)) & 1u; }
  __device__ __forceinline__ bool own_model(int i, int j) const { return ((model & own) >> (4 * i + j)) & 1u; }
  __device__ __forceinline__ int64_t gidx(const Dims& d, int i) const { return (int64_t)(z + i) * d.P + xs; }
  __device__ __forceinline__ int64_t midx(const Dims& d, int i, int j) const {
    return (int64_t)(z + i - d.N) * d.nx + (xs + j - d.mx0);
  }
  __device__ __forceinline__ void load(const Dims& d, const float* lev, float (&v)[PZ][4]) const {
#pragma unroll
    for (int i = 0; i < PZ; ++i) {
      float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (in[i]) q = *reinterpret_cast<const float4*>(lev + gidx(d, i));
      v[i][0] = q.x; v[i][1] = q.y; v[i][2] = q.z; v[i][3] = q.w;
    }
  }
  __device__ __forceinline__ void store(const Dims& d, float* lev, const float (&v)[PZ][4]) const {
#pragma unroll
    for (int i = 0; i < PZ; ++i)
      if (own_row(i))
        *reinterpret_cast<float4*>(lev + gidx(d, i)) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
  }
  __device__ __forceinline__ void put(float* lds, const float (&v)[PZ][4]) const {
#pragma unroll
    for (int i = 0; i < PZ; ++i)
      *reinterpret_cast<float4*>(lds + lo + i * RX) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
  }
  // free surface: the rows above the region's first mirror its first three
  // with the opposite sign about the zero row between them
  __device__ __forceinline__ void put_image(float* lds, const float (&v)[PZ][4]) const {
#pragma unroll
    for (int i = 0; i < PZ; ++i)
      if (lz + i < kRadius - 1)
        *reinterpret_cast<float4*>(lds + (kRadius - 2 - (lz + i)) * RX + lx) =
            make_float4(-v[i][0], -v[i][1], -v[i][2], -v[i][3]);
  }
  // zeros above and below the region
  __device__ __forceinline__ void clear_rim(float* lds) const {
    for (int k = threadIdx.x; k < 2 * kRadius * RX; k += NT) lds[k < kRadius * RX ? k : k + RZ * RX] = 0.0f;
  }
  // L u of the patch, in the z sweeps' order of operations.  The rows above
  // and below come from LDS, the columns beside it from the neighbouring
  // lanes (zero beyond the region).
  __device__ __forceinline__ void lap(const float* lds, const float (&c)[PZ][4], float (&out)[PZ][4]) const {
    const float* l = lds + lo;
    float col[PZ + 2 * kRadius][4];
#pragma unroll
    for (int r = 0; r < PZ + 2 * kRadius; ++r) {
      if (r >= kRadius && r < PZ + kRadius) {
#pragma unroll
        for (int j = 0; j < 4; ++j) col[r][j] = c[r - kRadius][j];
      } else {
        const float4 q = *reinterpret_cast<const float4*>(l + (r - kRadius) * RX);
        col[r][0] = q.x; col[r][1] = q.y; col[r][2] = q.z; col[r][3] = q.w;
      }
    }
#pragma unroll
    for (int i = 0; i < PZ; ++i) {
      float row[12];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        row[j] = from_lane<kDppRight1>(c[i][j]);
        row[4 + j] = c[i][j];
        row[8 + j] = from_lane<kDppLeft1>(c[i][j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = kRadius; k >= 1; --k) {
          const float sz = col[i + kRadius - k][j] + col[i + kRadius + k][j];
          const float sx = row[4 + j - k] + row[4 + j + k];
          acc = fmaf(bck(k), fmaf(-4.0f, c[i][j], sz + sx), acc);
        }
        out[i][j] = acc;
      }
    }
  }
};

// The patch's cells in the 4-cell ring around the model: cell (i, j) of the
// ring's sides has index sb + 4 i + j, of its top and bottom rows
// tb + nx i + j.  One base of each serves a patch because it never holds
// cells of both sides (patches start a multiple of 4 columns from the model's
// first one, so those that start left of the model end there) nor of top and
// bottom (a patch of four rows is not used on models of fewer than three).
struct Ring {
  int sb, tb;
  uint32_t side, rows;  // bits 4 i + j
  template <class P, int PZ>
  __device__ __forceinline__ void find(const P& p, const Dims& d, std::integral_constant<int, PZ>) {
    const int mz0 = p.z - d.N, mx0 = p.xs - d.mx0;
    side = rows = 0;
    sb = 8 * d.nx + 4 * mz0 + (mx0 < 0 ? mx0 + kRadius : 4 * d.nz + mx0 - d.nx);
    tb = mx0 + d.nx * (mz0 < 0 ? mz0 + kRadius : kRadius + mz0 - d.nz);
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int mz = mz0 + i, mx = mx0 + j;
        const uint32_t bit = 1u << (4 * i + j);
        if (!p.in[i]) continue;
        const bool zin = mz >= 0 && mz < d.nz, xin = mx >= 0 && mx < d.nx;
        if (zin && !xin && mx >= -kRadius && mx < d.nx + kRadius) side |= bit;
        if (xin && !zin && mz >= -kRadius && mz < d.nz + kRadius) rows |= bit;
      }
  }
  __device__ __forceinline__ Ring here() const {
    Ring q = *this;
    asm volatile("" : "+v"(q.sb), "+v"(q.tb), "+v"(q.side), "+v"(q.rows));
    return q;
  }
  // f(ring index of cell (i, j)) if it is in the ring
  template <class F>
  __device__ __forceinline__ void at(const Dims& d, int i, int j, F&& f) const {
    if (((side | rows) >> (4 * i + j)) & 1u) f((side >> (4 * i + j)) & 1u ? sb + 4 * i + j : tb + d.nx * i + j);
  }
};

// FP64 coefficients of the sponge by cells into it: 1 - g, 1 / (1 + g)
struct Sponge {
  double minus;
  Reciprocal plus;
};
__device__ __forceinline__ void sponge_table(Sponge* tab, double sp_a, int N) {
  for (int k = threadIdx.x; k <= N; k += blockDim.x) {
    const double gm = sp_a * (double)(k * k);
    tab[k] = Sponge{1.0 - gm, reciprocal(1.0 + gm)};
  }
}
// The damped cells of one row of a patch take ((1 - g) old + w lap) / (1 + g)
// (SECOND: (2 c - (1 - g) old + w lap) / (1 + g)) in FP64 instead of the plain
// update in v.  The division is quotient()'s.  Four cells at a time, so that their
// table reads and FP64 chains overlap.
template <bool SECOND>
__device__ __forceinline__ void damp_row(const Sponge (&t)[4], uint32_t model, const float (&c)[4],
                                         const float (&old)[4], const float (&w)[4], const float (&lap)[4],
                                         float (&v)[4]) {
  double x[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    x[j] = SECOND ? 2.0 * (double)c[j] - t[j].minus * (double)old[j] + (double)w[j] * (double)lap[j]
                  : t[j].minus * (double)old[j] + (double)w[j] * (double)lap[j];
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = quotient(x[j], t[j].plus);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float s = (float)x[j];
    asm volatile("" : "+v"(s));  // computed for every cell: no branch per cell
    v[j] = (model >> j) & 1u ? v[j] : s;
  }
}

// Receivers of the shot inside the region: slot -> (LDS offset, trace), at
// most kBlkRecv of them (the host sends no shot with more down this path).
template <int RX, int RZ>
__device__ __forceinline__ void list_receivers(const BlockArgs& a, const ShotDesc& sd, int cs0, int rz0, int x0, int x1,
                                               int z0, int z1, int* count, int* cell, int* trace, uint16_t* map) {
  for (int k = threadIdx.x; k < sd.nrec; k += blockDim.x) {
    const int2 c = a.rcell[sd.rec_begin + k];  // (padded row, storage column)
    if (c.x < z0 || c.x >= z1 || c.y < x0 || c.y >= x1) continue;
    const int s = atomicAdd(count, 1);
    const int lz = c.x - rz0, lx = c.y - cs0;
    if (cell) cell[s] = (lz + kRadius) * RX + lx;
    trace[s] = sd.rec_begin + k;
    if (map) map[lz * RX + lx] = (uint16_t)(s + 1);
  }
}

// -------------------------------------------------------------------------
// forward steps n0 = T q .. n0 + T - 1 of every shot of the batch, in the
// increment form of the z sweep
// -------------------------------------------------------------------------
template <int RX, int RZ, int PZ, int FLAGS>
__global__ __launch_bounds__(RX / 4 * (RZ / PZ), 4) void k_forward_block(BlockArgs a) {
  using PT = Patch<RX, RZ, PZ>;
  constexpr bool BORN = (FLAGS & kFwdBorn) != 0, CKPT = (FLAGS & kFwdCkpt) != 0, REC = (FLAGS & kFwdRecord) != 0;
  constexpr bool ILLUM = (FLAGS & kFwdIllum) != 0, CAP = (FLAGS & (kFwdCapD | kFwdCapU)) != 0;
  // two fields in turn take one barrier a step instead of two, where LDS is
  // not what limits the workgroups of a CU
  constexpr int NB = PZ == 1 || (PZ == 2 && !BORN) ? 2 : 1, SWAP = (NB - 1) * PT::LF;
  __shared__ __align__(16) float fu[NB * PT::LF];
  __shared__ __align__(16) float fb[BORN ? NB * PT::LF : 4];
  float *lu = fu, *lb = fb;
  __shared__ Sponge tab[kBlkSponge + 1];
  __shared__ int rcount, rcell[REC ? kBlkRecv : 1], rtrace[REC ? kBlkRecv : 1];
  __shared__ float wav[kBlkSteps];
  const StepArgs& s = a.s;
  const Dims& d = s.d;
  int slot, tile;
  map_block(a, slot, tile);
  const int bad = *s.err;
  const SlotInfo si = s.slots[slot];
  if (bad || si.shot < 0) return;
  const ShotDesc sd = s.shots[si.shot];
  const int q = s.step, n0 = q * a.T;
  const int ns = min(a.T, sd.nt - 1 - n0);
  if (ns <= 0) return;
  const PT p(a, d, tile);
  const int cs0 = p.xs - p.lx, rz0 = p.z - p.lz;
  const bool src_in = sd.src_z >= rz0 && sd.src_z < rz0 + RZ && sd.src_xs >= cs0 && sd.src_xs < cs0 + RX;
  // a region that the wavefield has not reached stays zero
  bool track = false;
  if (s.act) {
    const Reached r = reached(s, si.cs, rz0, rz0 + RZ, cs0, cs0 + RX, n0);
    if (!r.any && !src_in) {
      if constexpr (CAP) {  // the captured series of its cells
#pragma unroll
        for (int i = 0; i < PZ; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (p.own_model(i, j))
              for (int k = 0; k < ns; ++k)
                s.cap[((int64_t)slot * s.cap_T + (n0 + k - s.cap_n0)) * s.cap_R + p.midx(d, i, j)] = 0.0f;
      }
      return;
    }
    track = !r.all;
  }

  const int set_in = 3 * (q & 1), set_out = 3 - set_in;
  float* ubase = s.u + (int64_t)si.cs * s.ustride;
  float* bbase = BORN ? s.bu + (int64_t)si.cs * a.bstride : nullptr;
  float* E = ILLUM ? s.E + (int64_t)slot * d.model : nullptr;
  float uc[PZ][4], dn[PZ][4], w[PZ][4];
  float bc[BORN ? PZ : 1][4], bd[BORN ? PZ : 1][4], bw[BORN ? PZ : 1][4], ev[ILLUM ? PZ : 1][4];
  p.load(d, ubase + (int64_t)(set_in + (n0 & 1)) * d.field, uc);
  p.load(d, ubase + (int64_t)(set_in + 2) * d.field, dn);
  p.load(d, s.w, w);
  if constexpr (BORN) {
    p.load(d, bbase + (int64_t)(set_in + (n0 & 1)) * d.field, bc);
    p.load(d, bbase + (int64_t)(set_in + 2) * d.field, bd);
    p.load(d, s.bw, bw);
  }
  if constexpr (ILLUM) {
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) ev[i][j] = (n0 > 0 && p.own_model(i, j)) ? E[p.midx(d, i, j)] : 0.0f;
  }
  const float* wave = s.wavelet + (int64_t)si.shot * s.wstride;
  int src = -1;  // the source's cell in this patch
  if (src_in) {
    const int iz = sd.src_z - p.z, ix = sd.src_xs - p.xs;
    if (iz >= 0 && iz < PZ && ix >= 0 && ix < 4) src = 4 * iz + ix;
  }
  // (a scalar load inside the loop would make every LDS wait wait for it)
  if (src_in)
    for (int k = threadIdx.x; k < ns; k += PT::NT) wav[k] = wave[n0 + k];
  // the patch has owned cells in the ring around the model (whole workgroup: any patch)
  Ring ring;
  ring.side = ring.rows = 0;
  if constexpr (CKPT) {
    ring.find(p, d, std::integral_constant<int, PZ>{});
    ring.side &= p.own;
    ring.rows &= p.own;
  }
  bool sponge = false;
#pragma unroll
  for (int i = 0; i < PZ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) sponge |= !p.is_model(i, j);
  sponge = __any(sponge);  // per wavefront: some cell is not a plain interior one
  const bool image = d.fs && rz0 == d.ztop;

#pragma unroll
  for (int b = 0; b < NB; ++b) {
    p.clear_rim(fu + b * PT::LF);
    if constexpr (BORN) p.clear_rim(fb + b * PT::LF);
  }
  sponge_table(tab, s.sp_a, d.N);
  if (threadIdx.x == 0) rcount = 0;
  lds_barrier();
  if constexpr (REC)
    list_receivers<RX, RZ>(a, sd, cs0, rz0, p.own_x0, p.own_x1, p.own_z0, p.own_z1, &rcount, rcell, rtrace, nullptr);
  p.put(lu, uc);
  if (image) p.put_image(lu, uc);
  if constexpr (BORN) {
    p.put(lb, bc);
    if (image) p.put_image(lb, bc);
  }
  lds_barrier();
  const int nrec = REC ? rcount : 0;
  // One row of cells per thread leaves registers for its table entries, which
  // the steps of a launch otherwise read again from LDS (24 x 16, 2 shots, 400
  // steps: 214 -> 188 us, reverse 315 -> 290; 200 x 100: 14.5 -> 13.3 us a launch)
  constexpr bool REGTAB = PZ == 1 && !BORN;
  Sponge treg[4];
  if (REGTAB && sponge) p.sponge(d, tab, 0, treg);
  // u[n+1] is saved where nt-2-n is a positive multiple of K: `save` steps
  // from now, as pair `snap`
  int save = CKPT ? (sd.nt - 2 - n0) % sd.K : 0, snap = CKPT ? (sd.nt - 2 - n0) / sd.K - 1 : 0;

  for (int k = 0; k < ns; ++k) {
    const int n = n0 + k;
    float lap[PZ][4], blap[BORN ? PZ : 1][4];
    p.lap(lu, uc, lap);
    if constexpr (BORN) p.lap(lb, bc, blap);
    if (src >= 0) {
      const float f = wav[k];
#pragma unroll
      for (int i = 0; i < PZ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (src == 4 * i + j) lap[i][j] += f;
    }
    if constexpr (CKPT) {
      // the level before the last one, for the reverse sweep's start
      if (n == sd.nt - 2) p.here().store(d, ubase + (int64_t)(set_out + (n & 1)) * d.field, uc);
    }
    float un[PZ][4], bn[BORN ? PZ : 1][4];
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        un[i][j] = fmaf(w[i][j], lap[i][j], dn[i][j]);
        if constexpr (BORN) bn[i][j] = fmaf(w[i][j], fmaf(bw[i][j], lap[i][j], blap[i][j]), bd[i][j]);
        if constexpr (ILLUM) {
          const float D = w[i][j] * lap[i][j];
          ev[i][j] = fmaf(D, D, ev[i][j]);
        }
      }
    if (sponge) {
      const PT r = p.here();
#pragma unroll
      for (int i = 0; i < PZ; ++i) {
        Sponge tl[4];
        if constexpr (!REGTAB) r.sponge(d, tab, i, tl);
        const Sponge(&t)[4] = REGTAB ? treg : tl;
        damp_row<false>(t, r.model >> (4 * i), dn[i], dn[i], w[i], lap[i], un[i]);
        if constexpr (BORN) damp_row<false>(t, r.model >> (4 * i), bd[i], bd[i], w[i], blap[i], bn[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        dn[i][j] = un[i][j];
        un[i][j] = uc[i][j] + un[i][j];
        if constexpr (BORN) {
          bd[i][j] = bn[i][j];
          bc[i][j] = bc[i][j] + bn[i][j];
        }
      }
    if constexpr (CAP) {
      float* cap = s.cap + ((int64_t)slot * s.cap_T + (n - s.cap_n0)) * s.cap_R;
      const PT r = p.here();
#pragma unroll
      for (int i = 0; i < PZ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (r.own_model(i, j)) cap[r.midx(d, i, j)] = (FLAGS & kFwdCapD) ? w[i][j] * lap[i][j] : un[i][j];
    }
    if constexpr (CKPT) {
      if (ring.side | ring.rows) {
        float* strip = s.strip + (int64_t)si.cs * s.strip_stride + (int64_t)(n + 1) * d.ring;
        const Ring rr = ring.here();
#pragma unroll
        for (int i = 0; i < PZ; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) rr.at(d, i, j, [&](int ri) { strip[ri] = un[i][j]; });
      }
      if (save == 0 && snap >= 0) {
        float* sn0 = s.snap + (int64_t)si.cs * s.snap_stride + (int64_t)snap * 2 * d.model;
        const PT r = p.here();
#pragma unroll
        for (int i = 0; i < PZ; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (r.own_model(i, j)) {
              const int64_t mi = r.midx(d, i, j);
              sn0[mi] = un[i][j];
              sn0[d.model + mi] = uc[i][j];
            }
      }
      if (--save < 0) {
        save = sd.K - 1;
        --snap;
      }
    }
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) uc[i][j] = un[i][j];
    if constexpr (NB == 1) lds_barrier();  // every read of the step before its writes
    lu = fu + (k & 1 ? 0 : SWAP);
    if constexpr (BORN) lb = fb + (k & 1 ? 0 : SWAP);
    p.put(lu, uc);
    if (image) p.put_image(lu, uc);
    if constexpr (BORN) {
      p.put(lb, bc);
      if (image) p.put_image(lb, bc);
    }
    lds_barrier();
    if constexpr (REC) {
      float* tr = s.traces + (int64_t)(n + 1) * s.ntrace;
      for (int r = threadIdx.x; r < nrec; r += PT::NT) tr[rtrace[r]] = BORN ? lb[rcell[r]] : lu[rcell[r]];
    }
  }
  const PT r = p.here();
  if (track) {
#pragma unroll
    for (int i = 0; i < PZ; ++i) {
      uint32_t any = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        any |= __float_as_uint(uc[i][j]) | __float_as_uint(dn[i][j]);
        if constexpr (BORN) any |= __float_as_uint(bc[i][j]) | __float_as_uint(bd[i][j]);
      }
      // the first lane of each of the map's columns in a row of 16 lanes marks it
      const uint64_t nz = __ballot(any != 0u && r.own_row(i));
      const int l = threadIdx.x & 63, left = min((kActCols - (r.xs & (kActCols - 1))) / 4, 16 - (l & 15));
      if (((l & 15) == 0 || (r.xs & (kActCols - 1)) == 0) && (nz >> l & ((1u << left) - 1)))
        mark_reached(s, si.cs, r.z + i, r.xs, n0 + 1);
    }
  }
  r.store(d, ubase + (int64_t)(set_out + ((n0 + ns) & 1)) * d.field, uc);
  r.store(d, ubase + (int64_t)(set_out + 2) * d.field, dn);
  if constexpr (BORN) {
    r.store(d, bbase + (int64_t)(set_out + ((n0 + ns) & 1)) * d.field, bc);
    r.store(d, bbase + (int64_t)(set_out + 2) * d.field, bd);
  }
  if constexpr (ILLUM) {
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (r.own_model(i, j)) E[r.midx(d, i, j)] = ev[i][j];
  }
}

// -------------------------------------------------------------------------
// reverse steps m = nt-1 - T q down to m - T + 1, as the one-step z sweep:
// source wavefield from the strips and snapshots, damped adjoint step with
// the receivers' psi, g += lam D, E += D^2
// -------------------------------------------------------------------------
template <int RX, int RZ, int PZ, bool EXT, bool IMGU>
__global__ __launch_bounds__(RX / 4 * (RZ / PZ), 4) void k_reverse_block(BlockArgs a) {
  using PT = Patch<RX, RZ, PZ>;
  constexpr int NB = PZ == 1 ? 2 : 1, SWAP = (NB - 1) * PT::LF;  // (as in the forward sweep)
  __shared__ __align__(16) float fu[NB * PT::LF];
  __shared__ __align__(16) float fl[NB * PT::LF];
  float *lu = fu, *ll = fl;
  __shared__ Sponge tab[kBlkSponge + 1];
  __shared__ int rcount, rtrace[kBlkRecv];
  __shared__ __align__(8) uint16_t map[RX * RZ];
  __shared__ float psi[2][kBlkRecv];
  __shared__ float wav[kBlkSteps];
  __shared__ __align__(16) float le[RX * RZ];  // E (each cell its own thread's: registers are what this kernel lacks)
  const StepArgs& s = a.s;
  const Dims& d = s.d;
  int slot, tile;
  map_block(a, slot, tile);
  const int bad = *s.err;
  const SlotInfo si = s.slots[slot];
  if (bad || si.shot < 0) return;
  const ShotDesc sd = s.shots[si.shot];
  const int q = s.step, j0 = q * a.T, m0 = sd.nt - 1 - j0;
  const int ns = min(a.T, m0);
  if (ns <= 0) return;
  const PT p(a, d, tile);
  const int cs0 = p.xs - p.lx, rz0 = p.z - p.lz;
  // u[k] at level ubi + (k & 1), lam[k] at level lbi + (k & 1)
  const int ubi = 3 * (q & 1), ubo = 3 - ubi, lbi = 2 * (q & 1), lbo = 2 - lbi;
  float* ubase = s.u + (int64_t)si.cs * s.ustride;
  float* lbase = s.lam + (int64_t)slot * s.lstride;
  float* G = s.g + (int64_t)slot * d.model;
  float* E = s.E + (int64_t)slot * d.model;
  float uc[PZ][4], up[PZ][4], lc[PZ][4], lp[PZ][4], w[PZ][4], g[PZ][4];
  p.load(d, ubase + (int64_t)(ubi + ((m0 - 1) & 1)) * d.field, uc);
  p.load(d, ubase + (int64_t)(ubi + (m0 & 1)) * d.field, up);
  p.load(d, lbase + (int64_t)(lbi + ((m0 + 1) & 1)) * d.field, lc);
  p.load(d, lbase + (int64_t)(lbi + (m0 & 1)) * d.field, lp);
  p.load(d, s.w, w);
#pragma unroll
  for (int i = 0; i < PZ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool om = p.own_model(i, j);
      g[i][j] = om ? G[p.midx(d, i, j)] : 0.0f;
      le[(p.lz + i) * RX + p.lx + j] = (om && q > 0) ? E[p.midx(d, i, j)] : 0.0f;
    }
  const float* wave = s.wavelet + (int64_t)si.shot * s.wstride;
  const bool src_in = sd.src_z >= rz0 && sd.src_z < rz0 + RZ && sd.src_xs >= cs0 && sd.src_xs < cs0 + RX;
  int src = -1;
  if (src_in) {
    const int iz = sd.src_z - p.z, ix = sd.src_xs - p.xs;
    if (iz >= 0 && iz < PZ && ix >= 0 && ix < 4) src = 4 * iz + ix;
  }
  if (src_in)
    for (int k = threadIdx.x; k < ns; k += PT::NT) wav[k] = wave[m0 - 1 - k];
  Ring ring;
  ring.find(p, d, std::integral_constant<int, PZ>{});
  bool sponge = false, anymod = false;
#pragma unroll
  for (int i = 0; i < PZ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sponge |= !p.is_model(i, j);
      anymod |= p.is_model(i, j);
    }
  sponge = __any(sponge);
  anymod = __any(anymod);
  const bool image = d.fs && rz0 == d.ztop;

  // the receivers of the region: the map from cell to psi slot + 1
  const bool recs = sd.nrec > 0;
  bool rec = false;
  if (threadIdx.x == 0) rcount = 0;
  if (recs) {
#pragma unroll
    for (int i = 0; i < PZ; ++i)
      *reinterpret_cast<uint2*>(map + (p.lz + i) * RX + p.lx) = make_uint2(0u, 0u);
    lds_barrier();
    list_receivers<RX, RZ>(a, sd, cs0, rz0, cs0, cs0 + RX, rz0, rz0 + RZ, &rcount, nullptr, rtrace, map);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < PZ; ++i) {
      const uint2 mr = *reinterpret_cast<const uint2*>(map + (p.lz + i) * RX + p.lx);
      rec |= (mr.x | mr.y) != 0u;
    }
  }
  lds_barrier();
  const int nrec = rcount;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    p.clear_rim(fu + b * PT::LF);
    p.clear_rim(fl + b * PT::LF);
  }
  sponge_table(tab, s.sp_a, d.N);
  p.put(lu, uc);
  p.put(ll, lc);
  if (image) {
    p.put_image(lu, uc);
    p.put_image(ll, lc);
  }
  for (int r = threadIdx.x; r < nrec; r += PT::NT) psi[0][r] = s.traces[(int64_t)m0 * s.ntrace + rtrace[r]];
  lds_barrier();

  constexpr bool REGTAB = PZ == 1 && RZ == 32;
  Sponge treg[4];
  if (REGTAB && sponge) p.sponge(d, tab, 0, treg);
  // restarts at nt-1-m = K, 2K, ...: the next one `restart` steps from now,
  // from pair `snap`
  int restart = (sd.K - j0 % sd.K) % sd.K, snap = (j0 + sd.K - 1) / sd.K - 1;

  for (int k = 0; k < ns; ++k) {
    const int m = m0 - k;
    // snapshot restart: u[m], u[m-1] of the model cells come from the pair
    if (restart == 0 && snap >= 0 && snap < sd.nsnap) {
      const float* sn0 = s.snap + (int64_t)si.cs * s.snap_stride + (int64_t)snap * 2 * d.model;
      const PT r = p.here();
#pragma unroll
      for (int i = 0; i < PZ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (r.is_model(i, j)) {
            const int64_t mi = r.midx(d, i, j);
            up[i][j] = sn0[mi];
            uc[i][j] = sn0[d.model + mi];
          }
      p.put(lu, uc);  // (the last step's reads of lu are behind a barrier)
      if (image) p.put_image(lu, uc);
      lds_barrier();
    }
    if (--restart < 0) {
      restart = sd.K - 1;
      ++snap;
    }
    const bool hasS = m >= 3;
    float st[PZ][4];
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) st[i][j] = 0.0f;
    if (hasS && (ring.side | ring.rows)) {
      const float* strip = s.strip + (int64_t)si.cs * s.strip_stride + (int64_t)(m - 2) * d.ring;
      const Ring rr = ring.here();
#pragma unroll
      for (int i = 0; i < PZ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) rr.at(d, i, j, [&](int ri) { st[i][j] = strip[ri]; });
    }
    const bool more = k + 1 < ns;
    // the next step's psi, in flight during this one
    float pn[(kBlkRecv + PT::NT - 1) / PT::NT];
#pragma unroll
    for (int t = 0; t < (kBlkRecv + PT::NT - 1) / PT::NT; ++t) {
      const int r = threadIdx.x + t * PT::NT;
      pn[t] = (more && r < nrec) ? s.traces[(int64_t)(m - 1) * s.ntrace + rtrace[r]] : 0.0f;
    }
    float lap[PZ][4], ln[PZ][4];
    p.lap(ll, lc, lap);
    if (rec) {
      const float* ps = psi[k & 1];
#pragma unroll
      for (int i = 0; i < PZ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = map[(p.lz + i) * RX + p.lx + j];
          if (r) lap[i][j] += ps[r - 1];
        }
    }
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) ln[i][j] = fmaf(w[i][j], lap[i][j], 2.0f * lc[i][j] - lp[i][j]);
    if (sponge) {
      const PT r = p.here();
#pragma unroll
      for (int i = 0; i < PZ; ++i) {
        Sponge tl[4];
        if constexpr (!REGTAB) r.sponge(d, tab, i, tl);
        const Sponge(&t)[4] = REGTAB ? treg : tl;
        damp_row<true>(t, r.model >> (4 * i), lc[i], lp[i], w[i], lap[i], ln[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) lp[i][j] = lc[i][j];
    __builtin_amdgcn_sched_barrier(0);  // one field's window in registers at a time
    // D = w (L u[m-1] + f), u[m-2], g, E on the model cells
    float un[PZ][4];
    if (anymod) {
      p.lap(lu, uc, lap);
      if (src >= 0) {
        const float f = wav[k];
#pragma unroll
        for (int i = 0; i < PZ; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (src == 4 * i + j) lap[i][j] += f;
      }
      const PT x = EXT ? p.here() : p;
#pragma unroll
      for (int i = 0; i < PZ; ++i) {
        float4* const er = reinterpret_cast<float4*>(le + (p.lz + i) * RX + p.lx);
        float4 e4 = *er;
        float e[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float D = w[i][j] * lap[i][j];
          const float v = fmaf(w[i][j], lap[i][j], 2.0f * uc[i][j] - up[i][j]);
          g[i][j] = fmaf(ln[i][j], IMGU ? uc[i][j] : D, g[i][j]);
          e[j] = fmaf(D, D, e[j]);
          un[i][j] = p.is_model(i, j) ? v : st[i][j];
          if constexpr (EXT) {
            if (x.own_model(i, j)) {
              const int64_t xo = ((int64_t)slot * s.ext_T + (j0 + k) % s.ext_T) * d.model + x.midx(d, i, j);
              s.ext_lam[xo] = ln[i][j];
              s.ext_D[xo] = D;
            }
          }
          up[i][j] = uc[i][j];
        }
        *er = make_float4(e[0], e[1], e[2], e[3]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < PZ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          un[i][j] = st[i][j];
          up[i][j] = uc[i][j];
        }
    }
#pragma unroll
    for (int i = 0; i < PZ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uc[i][j] = un[i][j];
        lc[i][j] = ln[i][j];
      }
    if constexpr (NB == 1) lds_barrier();
    lu = fu + (k & 1 ? 0 : SWAP);
    ll = fl + (k & 1 ? 0 : SWAP);
    p.put(lu, uc);
    p.put(ll, lc);
    if (image) {
      p.put_image(lu, uc);
      p.put_image(ll, lc);
    }
#pragma unroll
    for (int t = 0; t < (kBlkRecv + PT::NT - 1) / PT::NT; ++t) {
      const int r = threadIdx.x + t * PT::NT;
      if (more && r < nrec) psi[(k + 1) & 1][r] = pn[t];
    }
    lds_barrier();
  }
  const int m1 = m0 - ns;  // state: u[m1 - 1], u[m1], lam[m1 + 1], lam[m1 + 2]
  const PT r = p.here();
  r.store(d, ubase + (int64_t)(ubo + ((m1 - 1) & 1)) * d.field, uc);
  r.store(d, ubase + (int64_t)(ubo + (m1 & 1)) * d.field, up);
  r.store(d, lbase + (int64_t)(lbo + ((m1 + 1) & 1)) * d.field, lc);
  r.store(d, lbase + (int64_t)(lbo + (m1 & 1)) * d.field, lp);
#pragma unroll
  for (int i = 0; i < PZ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (r.own_model(i, j)) {
        G[r.midx(d, i, j)] = g[i][j];
        E[r.midx(d, i, j)] = le[(r.lz + i) * RX + r.lx + j];
      }
}

template <int RX, int RZ, int PZ>
hipError_t forward_shape(const BlockArgs& a, int flags, hipStream_t s) {
  const dim3 grid((unsigned)(a.nbx * a.nbz * a.s.S)), block(RX / 4 * (RZ / PZ));
#define FWI_BLK(F) \
  case F: hipLaunchKernelGGL((k_forward_block<RX, RZ, PZ, F>), grid, block, 0, s, a); break;
  switch (flags) {
    FWI_BLK(kFwdRecord)
    FWI_BLK(kFwdRecord | kFwdCkpt)
    FWI_BLK(kFwdIllum)
    FWI_BLK(kFwdRecord | kFwdBorn)
    FWI_BLK(kFwdRecord | kFwdCkpt | kFwdBorn)
    FWI_BLK(kFwdCapD)
    FWI_BLK(kFwdCapU)
    default: return hipErrorInvalidValue;
  }
#undef FWI_BLK
  return hipGetLastError();
}

template <int RX, int RZ, int PZ>
hipError_t reverse_shape(const BlockArgs& a, int flags, hipStream_t s) {
  const dim3 grid((unsigned)(a.nbx * a.nbz * a.s.S)), block(RX / 4 * (RZ / PZ));
  switch (flags) {
    case 0: hipLaunchKernelGGL((k_reverse_block<RX, RZ, PZ, false, false>), grid, block, 0, s, a); break;
    case kRevExt: hipLaunchKernelGGL((k_reverse_block<RX, RZ, PZ, true, false>), grid, block, 0, s, a); break;
    case kRevImgU: hipLaunchKernelGGL((k_reverse_block<RX, RZ, PZ, false, true>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

bool bad_args(const BlockArgs& a) {
  return a.nbx < 1 || a.nbz < 1 || a.T < 1 || a.T > kBlkSteps || a.s.S < 1 || (int64_t)a.nbx * a.nbz * a.s.S > INT32_MAX || a.s.d.N > kBlkSponge || !a.rcell;
}

}  // namespace

hipError_t launch_forward_block(const BlockArgs& a, int flags, hipStream_t s) {
  if (bad_args(a)) return hipErrorInvalidValue;
  if ((flags & kFwdBorn) && (!a.s.bu || !a.s.bw)) return hipErrorInvalidValue;
  if ((flags & (kFwdCapD | kFwdCapU)) && !a.s.cap) return hipErrorInvalidValue;
  switch (a.shape) {
    case kBlkSmall: return forward_shape<64, 32, 1>(a, flags, s);
    case kBlkWide: return forward_shape<64, 64, 1>(a, flags, s);
    case kBlkPair: return forward_shape<64, 64, 2>(a, flags, s);
    case kBlkTall: return forward_shape<64, 64, 4>(a, flags, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_reverse_block(const BlockArgs& a, int flags, hipStream_t s) {
  if (bad_args(a)) return hipErrorInvalidValue;
  if ((flags & kRevExt) && (!a.s.ext_lam || !a.s.ext_D || a.s.ext_T < 1)) return hipErrorInvalidValue;
  switch (a.shape) {
    case kBlkSmall: return reverse_shape<64, 32, 1>(a, flags, s);
    case kBlkWide: return reverse_shape<64, 64, 1>(a, flags, s);
    case kBlkPair: return reverse_shape<64, 64, 2>(a, flags, s);
    default: return hipErrorInvalidValue;  // (four rows of both fields do not fit the registers)
  }
}

}  // namespace fwi
