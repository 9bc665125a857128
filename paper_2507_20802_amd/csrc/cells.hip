// cells.hip -- cell binning by counting sort and Verlet neighbour lists on
// gfx950, for the slots whose lists the host rebuilds.
//
// Steps (one launch each, all on the context stream):
//   grid   copy the host-chosen cell grid into the slot state
//   bin    fractional coordinates s = H^-1 r (Eq. 1 box); wrap r into the
//          primary cell (r -= H floor(s)); cell index; place in the cell from
//          an integer atomic count
//   scan   exclusive scan of the counts per slot (one workgroup per slot); the
//          counts are cleared for the next rebuild
//   scat   each atom to its place (order inside a cell arbitrary)
//   perm   each atom to its rank by id in its cell (gives a deterministic
//          order): positions, velocities, ids into scratch
//   back   copy back; inverse permutation; the slot's build state
//   list   per force tile (tiles.h): its segment and halo run table, then
//          per cell of it the atoms against the 3^dim neighbouring cells,
//          keeping every image pair within rc_ab + skin; tiles with an LDS halo get the packed list
//          (16-bit byte offsets 8 h of the neighbour's halo slot h), the
//          others the word list (j | image code << 24); engine.h
// Integer atomics only; the result does not depend on their order.
#include <hip/hip_runtime.h>

#include "cellgeom.h"
#include "kernels.h"
#include "tiles.h"

namespace aqs {

namespace {

// grid per slot: nc0, nc1, nc2, tile width, tiles, list mode
__global__ void k_rb_grid(RebuildArgs a, const int32_t* nc3) {
  const int r = blockIdx.x;
  if (threadIdx.x == 0 && r < a.nreps) {
    State* st = a.state + a.reps[r];
    const int32_t* q = nc3 + kGridInts * r;
    st->nc[0] = q[0];
    st->nc[1] = q[1];
    st->nc[2] = q[2];
    st->tiles_x = q[3];
    st->ntiles = q[4];
    st->list_mode = q[5];
  }
}

template <int D>
__global__ __launch_bounds__(kBlock) void k_rb_bin(RebuildArgs a) {
  const int2 bt = a.blocks[blockIdx.x];
  if (bt.x < 0) return;
  const Geom g = a.geom[bt.x];
  const State* st = a.state + bt.x;
  const int li = bt.y * kBlock + threadIdx.x;
  const bool live = li < g.n;
  const int64_t gi = g.atom_off + min(li, g.n - 1);
  const Box b = box_at(g, st->k);
  double4 p = a.pos4[gi];
  double s[3];
  frac(b, p.x, p.y, (D == 3) ? p.z : 0.0, s);
  const double nx = floor(s[0]), ny = floor(s[1]), nz = (D == 3) ? floor(s[2]) : 0.0;
  if (live && (nx != 0.0 || ny != 0.0 || nz != 0.0)) {
    // back into the box: r -= H n
    p.x -= nx * b.h00 + ny * b.h01;
    p.y -= (b.h10 == 0.0) ? ny * b.h11 : nx * b.h10 + ny * b.h11;
    if (D == 3) p.z -= nz * b.h22;
    a.pos4[gi] = p;
    if (a.alt4) {
      double4 q = a.alt4[gi];
      q.x -= nx * b.h00 + ny * b.h01;
      q.y -= (b.h10 == 0.0) ? ny * b.h11 : nx * b.h10 + ny * b.h11;
      if (D == 3) q.z -= nz * b.h22;
      a.alt4[gi] = q;
    }
  }
  int c3[3];
  const int nc[3] = {st->nc[0], st->nc[1], st->nc[2]};
  const int c = cell_of_pos<D>(b, nc, p, c3);
  // Its place among the cell's atoms, which the scatter uses (a second pass of
  // atomics there took 17 us for one replica of 32768 atoms, 64 for 16).  Atoms
  // in memory order mostly share their neighbour's cell: one atomic per run of
  // lanes in the same cell.
  const int lane = threadIdx.x % kWave;
  const int key = live ? c : -1;
  const int before = __shfl_up(key, 1, kWave);
  const bool head = lane == 0 || key != before;
  const unsigned long long heads = __ballot(head);
  const int start = kWave - 1 - __clzll((long long)(heads & (~0ull >> (kWave - 1 - lane))));
  const unsigned long long later = lane == kWave - 1 ? 0ull : heads & (~0ull << (lane + 1));
  int base = 0;
  if (live && head)
    base = atomicAdd(a.cell_count + g.cell_off + c,
                     (later ? __ffsll((long long)later) - 1 : kWave) - lane);
  base = __shfl(base, start, kWave);
  if (!live) return;
  a.cell_of[gi] = c;
  a.tid_[gi] = base + lane - start;
}

__global__ __launch_bounds__(1024) void k_rb_scan(RebuildArgs a) {
  const int rep = a.reps[blockIdx.x];
  const Geom g = a.geom[rep];
  const State* st = a.state + rep;
  const int ncell = st->nc[0] * st->nc[1] * st->nc[2];
  __shared__ int part[1024];
  const int T = blockDim.x;
  const int per = (ncell + T - 1) / T;
  const int c0 = threadIdx.x * per, c1 = min(ncell, c0 + per);
  int sum = 0;
  for (int c = c0; c < c1; ++c) sum += a.cell_count[g.cell_off + c];
  part[threadIdx.x] = sum;
  __syncthreads();
  // Hillis-Steele inclusive scan of the per-thread sums (integers: exact)
  for (int off = 1; off < T; off <<= 1) {
    const int v = (threadIdx.x >= off) ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  int run = (threadIdx.x == 0) ? 0 : part[threadIdx.x - 1];
  for (int c = c0; c < c1; ++c) {
    const int n = a.cell_count[g.cell_off + c];
    a.cell_start[g.cell_off + c] = run;
    a.cell_count[g.cell_off + c] = 0;   // for the next rebuild
    run += n;
  }
  if (threadIdx.x == T - 1) a.cell_start[g.cell_off + ncell] = part[T - 1];
}

__global__ __launch_bounds__(kBlock) void k_rb_scatter(RebuildArgs a) {
  const int2 bt = a.blocks[blockIdx.x];
  if (bt.x < 0) return;
  const Geom g = a.geom[bt.x];
  const int li = bt.y * kBlock + threadIdx.x;
  if (li >= g.n) return;
  const int64_t gi = g.atom_off + li;
  const int c = a.cell_of[gi];
  a.order[g.atom_off + a.cell_start[g.cell_off + c] + a.tid_[gi]] = li;
}

// Atoms of a cell by id, moved to their new places, a lane per atom: its new
// place is its rank among the cell's ids (ids are distinct).  A wavefront per cell
// with the ids in LDS takes as long where cells are full (7.6 us for 32768 atoms in
// 3D, 31 against 35 for 16 of them) and is mostly idle where they are not: 87 us,
// now 7, for 159048 atoms in 2D at 0.8 per cell.
template <int D>
__global__ __launch_bounds__(kBlock) void k_rb_perm(RebuildArgs a) {
  const int2 bt = a.blocks[blockIdx.x];
  if (bt.x < 0) return;
  const Geom g = a.geom[bt.x];
  const int li = bt.y * kBlock + threadIdx.x;
  if (li >= g.n) return;
  const int64_t go = g.atom_off + li;
  const int32_t* o = a.order + g.atom_off;
  const int32_t* id = a.id + g.atom_off;
  const int c = a.cell_of[go], key = id[li];
  const int b = a.cell_start[g.cell_off + c], e = a.cell_start[g.cell_off + c + 1];
  int r = 0;
#pragma unroll 8
  for (int q = b; q < e; ++q) r += (id[o[q]] < key) ? 1 : 0;
  const int64_t gi = g.atom_off + b + r;
  a.tpos4[gi] = a.pos4[go];
  a.tvx[gi] = a.vx[go];
  a.tvy[gi] = a.vy[go];
  if (D == 3) a.tvz[gi] = a.vz[go];
  a.tid_[gi] = key;
  if (a.dlx) {
    a.tdlx[gi] = a.dlx[go];
    a.tdly[gi] = a.dly[go];
    if (D == 3) a.tdlz[gi] = a.dlz[go];
  }
  if (a.alt4) a.talt4[gi] = a.alt4[go];
}

template <int D>
__global__ __launch_bounds__(kBlock) void k_rb_back(RebuildArgs a) {
  const int2 bt = a.blocks[blockIdx.x];
  if (bt.x < 0) return;
  const Geom g = a.geom[bt.x];
  const int li = bt.y * kBlock + threadIdx.x;
  if (threadIdx.x == 0) {
    a.upart[g.block0 + bt.y] = 0.0;   // no displacement since this build
    if (bt.y == 0) {
      State* st = a.state + bt.x;
      st->ubound = 0.0;
      st->gamma_build = strain_of(st->k, g.dgamma);
      st->k_build = st->k;
      if (a.resume && st->phase == PH_REBUILD)
        st->phase = (st->resume_phase == PH_LPLAIN || st->resume_phase == PH_LMOVE ||
                     st->resume_phase == PH_LREVERT || st->resume_phase == PH_CG)
                        ? st->resume_phase
                        : PH_FIRE;
    }
  }
  if (li >= g.n) return;
  const int64_t gi = g.atom_off + li;
  a.pos4[gi] = a.tpos4[gi];
  a.xref4[gi] = a.tpos4[gi];
  a.vx[gi] = a.tvx[gi];
  a.vy[gi] = a.tvy[gi];
  if (D == 3) a.vz[gi] = a.tvz[gi];
  const int32_t aid = a.tid_[gi];
  a.id[gi] = aid;
  a.inv[g.atom_off + aid] = li;
  if (a.dlx) {
    a.dlx[gi] = a.tdlx[gi];
    a.dly[gi] = a.tdly[gi];
    if (D == 3) a.dlz[gi] = a.tdlz[gi];
  }
  if (a.alt4) a.alt4[gi] = a.talt4[gi];
}

// Neighbour lists, one block per force tile (tiles.h).  The tile's segment and
// candidate runs are computed here.  A cell's atoms share their candidates:
// per neighbouring row one contiguous range of candidate numbers (the wrapped
// cells' runs are numbered next to their row's), 3 or 9 ranges that a cell
// numbers on its own, in chunks of 64.
//   test     a wavefront takes up to kUnitAtoms atoms of one cell and walks
//            the cell's chunks, one candidate per lane (loaded a chunk ahead
//            and turned into an FP32 offset from the tile's first atom), the
//            atoms one after another: the ballot of the distance test is the
//            atom's neighbour mask of the chunk, kept in LDS.  Every
//            candidate that some mask names is flagged.
//   number   the flagged candidates in order form the compact halo (stored for
//            the force kernel as j | code << 24) and their bit counts give each
//            its halo slot.
//   write    a lane takes half of the A or of the B neighbours of one atom in the tile's
//            walk order, turns its masks' bits into byte offsets of halo slots
//            through the cell's table and stores whole groups; the lanes of a
//            wavefront store neighbouring columns.
// The test is bound by its vector instructions: about 12 per atom and chunk,
// 64 pairs.  One candidate per lane keeps every lane busy, where a lane per atom
// left over half of the block idle, read each candidate from LDS once for
// every atom and sent each entry to memory twice, one by one.  Rebuild of 16 x
// 32768 atoms (3D, 16 of them at once): 497 us, 2156 before; of one replica 55,
// 197 before.
// "Cell" above is a group of neighbouring cells of the row where a tile spans
// more of them than the tables below hold (short cutoffs, tiles filled to the
// limit): the group's atoms share the candidates around it.
// A tile whose compact halo does not fit in the force kernel's LDS gets word
// lists (j | code); so does a tile past the limits below, tested in FP64
// straight from the cells (kernel's end), and a wide tile of a slot with fewer
// than two atoms per cell.  There the halo hardly shortens a force launch, and
// the search takes less time: 2D, 159048 atoms, cutoff 2.5, list kernel and mean
// force launch, groups against search: 92 and 11.0 us, 61 and 10.9 at 0.8 atoms
// per cell; 88 and 8.1 us, 50 and 9.5 at 2.4, where lists that live over about 25
// iterations pay for the groups.
// Times below: a rebuild's list kernel for 32768 atoms in 3D and for 16 of them,
// 54.6 and 497 us as it is.
constexpr int kListBlock = 512;     // threads of the list kernel (256: 68 and 673)
// A unit's chunks are split over this many wavefronts.  1: 54.4 and 479, but 158
// instead of 146 for one replica of 132651 atoms; 4: 55 and 510, and in 2D 24
// instead of 20.5 for 4 x 2116 atoms.
constexpr int kChunkParts = 2;
// Atoms of one cell that a wavefront tests together: 8: 64 and 566; 32: 48 and 446.
constexpr int kUnitAtoms = 16;
// What the tables in LDS hold: a glass's tiles in 3D span 4 to 15 cells of about
// 11 chunks, in 2D 12 to 25 cells of 2 chunks; two blocks per CU, which the
// registers allow, fit with them.
constexpr int kListCells = 96;      // groups of cells in a tile
constexpr int kTileChunks = 128;    // chunks of all their candidates
// Cells of a group at first (the chunks may ask for four times as many): FP32
// offsets within it, a few hundred list distances, round far below kListMargin.
// A tile of more cells than 96 such groups goes to the FP64 search.
constexpr int kGroupCells = 128;
static_assert(kTileChunks >= kCandCap / kWave, "one group of all candidates fits");
// Masks kept at once; larger tiles go in batches of atoms, tested twice (1024: 94 and
// 634; 4096: as it is).
constexpr int kMaskWords = 2048;

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ int wave_scan(int v) {
  const int lane = threadIdx.x % kWave;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(v, o, kWave);
    if (lane >= o) v += u;
  }
  return v;
}

// Counts v[0 .. n - 1] to their exclusive sums v[0 .. n], n <= kListCells, by
// one wavefront.
__device__ __forceinline__ void scan_cells(uint16_t* v, int n) {
  static_assert(kListCells <= 2 * kWave, "two cells per lane");
  const int lane = threadIdx.x % kWave;
  const int c0 = 2 * lane < n ? v[2 * lane] : 0, c1 = 2 * lane + 1 < n ? v[2 * lane + 1] : 0;
  const int before = wave_scan(c0 + c1) - (c0 + c1);
  if (2 * lane <= n) v[2 * lane] = (uint16_t)before;
  if (2 * lane + 1 <= n) v[2 * lane + 1] = (uint16_t)(before + c0);
  if (lane == kWave - 1 && n == 2 * kWave) v[n] = (uint16_t)(before + c0 + c1);
}

template <int D>
__global__ __launch_bounds__(kListBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_rb_list(RebuildArgs a) {
  const int2 bt = a.tiles[blockIdx.x];
  if (bt.x < 0) return;
  const State* st = a.state + bt.x;
  if (bt.y >= st->ntiles) return;
  const Geom g = a.geom[bt.x];
  const Box bx = box_at(g, st->k);
  const int nc[3] = {st->nc[0], st->nc[1], st->nc[2]};
  const int32_t* cs = a.cell_start + g.cell_off;
  const double4* P = a.pos4 + g.atom_off;
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  constexpr int CAP = (D == 3) ? kHaloCap3 : kHaloCap2;
  constexpr int R = (D == 3) ? 9 : 3;        // neighbouring rows of a cell
  constexpr int R0 = (D == 3) ? 0 : 3;       // first of them among the runs' rows
  constexpr int NW = kListBlock / kWave;
  __shared__ TileRun runs[kRuns];
  __shared__ double s_sh[kRuns][3];          // image shifts
  __shared__ int s_c0[kRuns / 3];            // first cell of each neighbouring row
  __shared__ int s_cx0, s_cx1, s_ncand, s_words, s_halo;
  __shared__ int s_cs[kListCells + 1];       // first atom of each cell of the tile
  __shared__ uint16_t s_lo[kListCells][R];   // a cell's ranges: first candidate
  __shared__ uint16_t s_p[kListCells][R + 1];  // ... and its number within the cell
  __shared__ uint16_t s_cb[kListCells + 1];  // first chunk of each cell
  __shared__ uint16_t s_uo[kListCells + 1];  // first unit of each cell
  __shared__ unsigned long long s_mask[kMaskWords];
  __shared__ unsigned long long s_ta[kTileChunks];   // candidates of type A
  __shared__ uint16_t s_map[kTileChunks * kWave];    // candidate, then byte offset of its halo slot
  __shared__ __align__(8) uint8_t s_flag[kCandCap];  // candidates named by some list
  __shared__ unsigned long long s_bits[kCandCap / kWave];
  __shared__ int s_pre[kCandCap / kWave];
  __shared__ float4 s_atom[NW][kUnitAtoms];  // the atoms of each wavefront's unit
  __shared__ int s_cnt0[kTileSort];          // list counts in tile order
  __shared__ uint16_t s_rank[kTileSort];     // walk order: rank of an atom, then (s_src) atom of a rank
  __shared__ uint16_t s_src[kTileSort];
  __shared__ uint8_t s_cell[kTileSort];      // cell of an atom
  int a0, a1, cy, cz;
  segment(nc, st->tiles_x, cs, bt.y, a0, a1, cy, cz);
  const int nt = a1 - a0;
  const int64_t tix = g.tile_off + bt.y;
  const int row0 = (cz * nc[1] + cy) * nc[0];
  if (tid == 0) {
    s_cx0 = 0;
    s_cx1 = 0;
  }
  __syncthreads();
  if (nt > 0 && nc[0] <= kListBlock) {
    if (tid < nc[0]) {
      const int b = cs[row0 + tid], e = cs[row0 + tid + 1];
      if (b <= a0 && a0 < e) s_cx0 = tid;
      if (b < a1 && a1 <= e) s_cx1 = tid;
    }
  } else if (nt > 0 && tid < 2) {   // a longer row: where its first and last atom were binned
    int c3[3];
    cell_of_pos<D>(bx, nc, P[tid == 0 ? a0 : a1 - 1], c3);
    (tid == 0 ? s_cx0 : s_cx1) = c3[0];
  }
  __syncthreads();
  const int cx0 = s_cx0, row_cells = s_cx1 - s_cx0 + 1;
  if (tid < kRuns) {
    runs[tid] = make_run<D>(tid, cx0, s_cx1, cy, cz, nc, cs);
    code_shift(tid, bx, s_sh[tid]);
  }
  if (tid < kRuns / 3) {
    const int ry = cy + tid % 3 - 1, rz = (D == 3) ? cz + tid / 3 - 1 : 0;
    const int y = ry < 0 ? ry + nc[1] : (ry >= nc[1] ? ry - nc[1] : ry);
    const int z = rz < 0 ? rz + nc[2] : (rz >= nc[2] ? rz - nc[2] : rz);
    s_c0[tid] = (z * nc[1] + y) * nc[0];
  }
  for (int i = tid; i < min(nt, kTileSort); i += kListBlock) s_cnt0[i] = 0;
  for (int h = tid; h < kCandCap / 8; h += kListBlock) reinterpret_cast<uint64_t*>(s_flag)[h] = 0u;
  __syncthreads();
  if (wv == 0) {
    const int c = lane < kRuns ? runs[lane].count : 0;
    const int inc = wave_scan(c);
    if (lane < kRuns) runs[lane].off = inc - c;
    if (lane == kWave - 1) {
      s_ncand = inc;
      s_words = 0;
    }
  }
  __syncthreads();
  const int ncand = s_ncand;
  const bool fast = st->list_mode == 0 && ncand <= kCandCap && nt <= kTileSort &&
                    (row_cells <= kListCells ||
                     (g.n >= 2 * nc[0] * nc[1] * nc[2] && row_cells <= kListCells * kGroupCells));
  // The groups' ranges: groups of one cell, mostly; of as many as it takes for the
  // tables to hold them and their chunks (a single group's always fit).
  int gw = 1, ncell = 1;
  if (row_cells > kListCells)   // ... and about a unit's atoms each, whose candidates mostly fit in one chunk
    gw = max((row_cells + kListCells - 1) / kListCells,
             min(kGroupCells, (kUnitAtoms * row_cells + nt - 1) / max(nt, 1)));
  while (fast) {
    ncell = (row_cells + gw - 1) / gw;
    for (int ci = tid; ci <= ncell; ci += kListBlock) s_cs[ci] = cs[row0 + cx0 + min(ci * gw, row_cells)];
    for (int e = tid; e < ncell * R; e += kListBlock) {
      const int ci = e / R, q = e % R, r = 3 * (q + R0), c0 = s_c0[q + R0];
      const int cx = cx0 + ci * gw, cl = cx0 + min((ci + 1) * gw, row_cells) - 1;   // its first and last cell
      const TileRun m = runs[r + 1];
      s_lo[ci][q] = (uint16_t)(cx > 0 ? m.off + (cs[c0 + cx - 1] - m.src) : runs[r].off);
      const int hi = cl + 1 < nc[0] ? m.off + (cs[c0 + cl + 2] - m.src) : runs[r + 2].off + runs[r + 2].count;
      s_p[ci][q + 1] = (uint16_t)(hi - s_lo[ci][q]);
    }
    __syncthreads();
    for (int ci = tid; ci < ncell; ci += kListBlock) {
      int acc = 0;
      s_p[ci][0] = 0;
      for (int q = 1; q <= R; ++q) {
        acc += s_p[ci][q];
        s_p[ci][q] = (uint16_t)acc;
      }
      const bool any = min(s_cs[ci + 1], a1) > max(s_cs[ci], a0);   // atoms of the tile in the cell
      const int ch = any ? (acc + kWave - 1) / kWave : 0;
      s_cb[ci] = (uint16_t)ch;
      atomicMax(&s_words, ch);
    }
    __syncthreads();
    if (wv == 0) scan_cells(s_cb, ncell);
    __syncthreads();
    if (s_cb[ncell] <= kTileChunks) break;
    gw = min(2 * gw, row_cells);
    __syncthreads();
    if (tid == 0) s_words = 0;
    __syncthreads();
  }
  const int words = max(s_words, 1);
  const double4 ref = nt > 0 ? P[a0] : make_double4(0.0, 0.0, 0.0, 0.0);
  const int batch = max(1, min(nt, kMaskWords / words));   // atoms whose masks fit at once
  const int G = a.max_nb / kGroup;
  if (fast) {
    // list distance (squared, with the margin) of an atom's type t and a candidate's type
    float thr[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double rc = sqrt(a.pp[2 * t + u].rc2) + a.skin;
        thr[t][u] = (float)((rc + kListMargin) * (rc + kListMargin));
      }
    // j | image code of a candidate
    auto global_entry = [&](int hc) {
      int r = R0;   // its row: the last that starts no later
#pragma unroll
      for (int k = 1; k < R; ++k) r += runs[3 * (R0 + k)].off <= hc ? 1 : 0;
      const TileRun m = runs[3 * r + 1];
      const TileRun rr = runs[3 * r + (hc >= m.off ? 1 : 0) + (hc >= m.off + m.count ? 1 : 0)];
      return (uint32_t)(rr.src + (hc - rr.off)) | ((uint32_t)rr.code << kCodeShift);
    };
    auto slot_of = [&](int hc) {
      const int w = hc / kWave;
      return s_pre[w] + __popcll(s_bits[w] & ((1ull << (hc % kWave)) - 1ull));
    };
    constexpr uint32_t fill = 8u * (uint32_t)(CAP - 1);
    bool lds = true;
    // Steps 0 .. nbatch - 1 test the atoms, a batch each (counts, candidate tables
    // and flags with them), the last of them numbers the candidates, and
    // the steps after it write the lists (of several batches, tested again first).
    const int nbatch = max(1, (nt + batch - 1) / batch);
    for (int step = 0; step < 2 * nbatch; ++step) {
      const bool first = step < nbatch;
      const int b0 = (step % nbatch) * batch, b1 = min(nt, b0 + batch);
      __syncthreads();
      if (first || nbatch > 1) {
        for (int ci = tid; ci < ncell; ci += kListBlock)
          s_uo[ci] = (uint16_t)(max(0, min(s_cs[ci + 1], a0 + b1) - max(s_cs[ci], a0 + b0) + kUnitAtoms - 1) /
                                kUnitAtoms);
        __syncthreads();
        if (wv == 0) scan_cells(s_uo, ncell);
        __syncthreads();
        const int nunit = s_uo[ncell];
        for (int item = wv; item < kChunkParts * nunit; item += NW) {
          const int u = item / kChunkParts;
          // the unit's cell: the last whose first unit is not past u
          int ci = -1;
          for (int c0 = 0; c0 < ncell; c0 += kWave)
            ci += __popcll(__ballot(c0 + lane < ncell && (int)s_uo[c0 + lane] <= u));
          ci = __builtin_amdgcn_readfirstlane(ci);
          // the cell's atoms in nearly equal units
          const int y0 = max(s_cs[ci], a0 + b0), y1 = min(s_cs[ci + 1], a0 + b1);
          const int uc = u - (int)s_uo[ci], nu = (int)s_uo[ci + 1] - (int)s_uo[ci];
          const int x0 = y0 + uc * (y1 - y0) / nu;
          const int cnt = __builtin_amdgcn_readfirstlane(y0 + (uc + 1) * (y1 - y0) / nu - x0);
          const int total = __builtin_amdgcn_readfirstlane(s_p[ci][R]), cb = s_cb[ci];
          const int nch = (total + kWave - 1) / kWave;
          // this item's share of the chunks
          const int ch0 = item % kChunkParts * nch / kChunkParts,
                    ch1 = (item % kChunkParts + 1) * nch / kChunkParts;
          if (ch0 == ch1) continue;
          // the cell's tables are written by the first unit that sees the cell
          const bool tables = first && x0 == max(s_cs[ci], a0);
          // lane q < cnt: atom x0 + q, its own number among the cell's candidates
          int aw = 0;
          int na = 0, nb = 0;
          float4 at = make_float4(1e18f, 0.f, 0.f, 0.f);   // past the unit: no candidate is near
          const double4 from = gw > 1 ? P[x0] : ref;       // a tile of wide groups is long
          if (lane < cnt) {
            const double4 pi = P[x0 + lane];
            at.x = (float)(pi.x - from.x);
            at.y = (float)(pi.y - from.y);
            at.z = (D == 3) ? (float)(pi.z - from.z) : 0.0f;
            at.w = (float)pi.w;
            constexpr int q0 = R / 2;            // the atom's own row
            const TileRun m = runs[3 * (q0 + R0) + 1];
            const int own = m.off + (x0 + lane - m.src) - (int)s_lo[ci][q0] + (int)s_p[ci][q0];
            aw = own;
            if (first) s_cell[x0 + lane - a0] = (uint8_t)ci;
          }
          if (lane < kUnitAtoms) s_atom[wv][lane] = at;
          int sp[R];
#pragma unroll
          for (int q = 1; q < R; ++q) sp[q] = s_p[ci][q];
          // this lane's candidate of chunk ch, loaded
          auto load = [&](int ch, int& hc, int& code, double4& pj) {
            const int p = ch * kWave + lane;
            int q = 0;   // the range that holds number p
#pragma unroll
            for (int k = 1; k < R; ++k) q += p >= sp[k] ? 1 : 0;
            hc = p < total ? p + (int)s_lo[ci][q] - (int)s_p[ci][q] : -1;
            if (hc >= 0) {
              const int r = 3 * (q + R0);
              const TileRun m = runs[r + 1];
              const TileRun rr = runs[r + (hc >= m.off ? 1 : 0) + (hc >= m.off + m.count ? 1 : 0)];
              code = rr.code;
              pj = P[rr.src + (hc - rr.off)];
            }
          };
          int hc_n = -1, code_n = 13;
          double4 pj_n = make_double4(0.0, 0.0, 0.0, 0.0);
          load(ch0, hc_n, code_n, pj_n);
          for (int ch = ch0; ch < ch1; ++ch) {
            const int hc = hc_n, code = code_n;
            const double4 pj = pj_n;
            if (ch + 1 < ch1) load(ch + 1, hc_n, code_n, pj_n);
            const float px = (float)((pj.x + s_sh[code][0]) - from.x);
            const float py = (float)((pj.y + s_sh[code][1]) - from.y);
            const float pz = (D == 3) ? (float)((pj.z + s_sh[code][2]) - from.z) : 0.0f;
            const bool tb = pj.w != 0.0;
            // a lane without a candidate passes no test
            const float t0 = hc < 0 ? -1.0f : (tb ? thr[0][1] : thr[0][0]);
            const float t1 = hc < 0 ? -1.0f : (tb ? thr[1][1] : thr[1][0]);
            unsigned long long any = 0ull;
            unsigned long long mine = 0ull;   // lane q: the mask of atom q
            for (int q0 = 0; q0 < cnt; q0 += 4) {
              float4 x[4];
#pragma unroll
              for (int q = 0; q < 4; ++q) x[q] = s_atom[wv][q0 + q];
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const float fx = px - x[q].x, fy = py - x[q].y, fz = (D == 3) ? pz - x[q].z : 0.0f;
                const float t = x[q].w != 0.0f ? t1 : t0;
                const unsigned long long m = __ballot(fx * fx + fy * fy + fz * fz < t);
                any |= m;
                mine = lane == q0 + q ? m : mine;
              }
            }
            const unsigned long long ta = __ballot(hc >= 0 && !tb);
            if (lane < cnt) {
              if (aw / kWave == ch) mine &= ~(1ull << (aw % kWave));   // not its own neighbour
              s_mask[(x0 - a0 - b0 + lane) * words + ch] = mine;
              na += __popcll(mine & ta);
              nb += __popcll(mine & ~ta);
            }
            if (first) {
              if ((any >> lane) & 1ull) s_flag[hc] = 1;
              if (tables) {
                s_map[(cb + ch) * kWave + lane] = (uint16_t)max(hc, 0);
                if (lane == 0) s_ta[cb + ch] = ta;
              }
            }
          }
          if (first && lane < cnt) atomicAdd(&s_cnt0[x0 - a0 + lane], na | (nb << 16));
        }
        __syncthreads();
      }
      if (first) {
        if (step < nbatch - 1) continue;
        for (int i = tid; i < nt; i += kListBlock) {
          // both segments' groups have to fit side by side in the packed list
          const int na = s_cnt0[i] & 0xffff, nb = s_cnt0[i] >> 16;
          if (na + nb > a.max_nb || (na + kGroup - 1) / kGroup + (nb + kGroup - 1) / kGroup > G) {
            atomicMax(a.overflow, na + nb);
            s_cnt0[i] = 0;
          }
        }
        // number the flagged candidates
        const int nw = (ncand + kWave - 1) / kWave;
        for (int w = wv; w < nw; w += NW) {
          const int h = w * kWave + lane;
          const unsigned long long m = __ballot(h < ncand && s_flag[h] != 0);
          if (lane == 0) s_bits[w] = m;
        }
        __syncthreads();
        if (wv == 0) {
          const int c = lane < nw ? __popcll(s_bits[lane]) : 0;
          const int inc = wave_scan(c);
          if (lane < nw) s_pre[lane] = inc - c;
          if (lane == kWave - 1) s_halo = inc;
        }
        __syncthreads();
        // LDS halo slot CAP - 1 is the force kernel's far fill slot
        const int halo = s_halo;
        lds = halo < CAP;
        if (tid == 0) {
          TileHdr h;
          h.a0 = a0;
          h.a1 = a1;
          h.pad_ = 0;
          h.halo = lds ? halo : -1;
          a.thdr[tix] = h;
        }
        if (lds) {
          uint32_t* hx = a.hidx + tix * CAP;
          for (int hc = tid; hc < ncand; hc += kListBlock)
            if (s_flag[hc]) hx[slot_of(hc)] = global_entry(hc);
          for (int e = tid; e < s_cb[ncell] * kWave; e += kListBlock)
            s_map[e] = (uint16_t)(8 * slot_of(s_map[e]));
        }
        // Walk order.  The consumers of a tile with an LDS halo walk its atoms by
        // decreasing list length (ties by position), so the lanes of a wavefront
        // have lists of similar length: tord[a0 + k] is the k-th atom, and its
        // packed list and count sit in column a0 + k, so a wavefront still reads
        // consecutive list words.  Other tiles keep their atoms in tile order.
        for (int i = tid; i < nt; i += kListBlock) {
          const int ci = (s_cnt0[i] & 0xffff) + (s_cnt0[i] >> 16);
          int rank = i;
          if (lds) {
            rank = 0;
            for (int k = 0; k < nt; ++k) {
              const int cj = (s_cnt0[k] & 0xffff) + (s_cnt0[k] >> 16);
              rank += (cj > ci || (cj == ci && k < i)) ? 1 : 0;
            }
          }
          s_rank[i] = (uint16_t)rank;
          s_src[rank] = (uint16_t)i;
          a.tord[g.atom_off + a0 + rank] = a0 + i;
          a.nbc[g.atom_off + a0 + rank] = s_cnt0[i];
        }
        __syncthreads();
        continue;
      }
      const int bn = b1 - b0;
      // an item: half of the A or of the B neighbours of an atom, whole groups
      for (int e = tid; e < 4 * bn; e += kListBlock) {
        const bool isa = e < 2 * bn;
        const int k = (e % (2 * bn)) % bn, half = (e % (2 * bn)) / bn;
        // all masks present: columns in walk order; a batch: atoms in tile order
        const int i = nbatch > 1 ? b0 + k : (int)s_src[k];
        const int col = s_rank[i];
        const int cb = s_cb[s_cell[i]];
        const unsigned long long* M = s_mask + (i - b0) * words;
        const int n = isa ? (s_cnt0[i] & 0xffff) : (s_cnt0[i] >> 16);
        const int ng = (n + kGroup - 1) / kGroup;
        const int g0 = half ? (ng + 1) / 2 : 0, g1 = half ? ng : (ng + 1) / 2;
        if (g0 == g1) continue;
        auto word = [&](int w) {   // (past the last word: not used)
          w = min(w, words - 1);
          const unsigned long long ta = s_ta[min(cb + w, kTileChunks - 1)];
          return M[w] & (isa ? ta : ~ta);
        };
        // the half's first neighbour
        int w = 0, skip = kGroup * g0;
        unsigned long long m = word(0);
        for (int c = __popcll(m); c <= skip; c = __popcll(m)) {
          skip -= c;
          m = word(++w);
        }
        for (; skip > 0; --skip) m &= m - 1ull;
        unsigned long long ahead = word(w + 1);
        auto next = [&]() -> uint32_t {   // the map entry of the segment's next neighbour
          while (m == 0ull) {
            m = ahead;
            ++w;
            ahead = word(w + 1);
          }
          const int bit = __ffsll((long long)m) - 1;
          m &= m - 1ull;
          return s_map[(cb + w) * kWave + bit];
        };
        if (lds) {
          uint2* Pk = a.nbp + g.nb_off / kGroup + a0 + col;
          for (int gs = g0; gs < g1; ++gs) {
            uint32_t o[kGroup];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) o[q] = kGroup * gs + q < n ? next() : fill;
            Pk[(int64_t)(isa ? gs : G - 1 - gs) * g.npad] =
                make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
          }
        } else {
          uint32_t* L = a.nbl + g.nb_off + a0 + col;
          for (int q = kGroup * g0; q < min(kGroup * g1, n); ++q)
            L[(int64_t)(isa ? q : a.max_nb - 1 - q) * g.npad] = global_entry((int)next());
        }
      }
    }
    return;
  }
  // A tile past the limits (or lists asked for as words): each atom scans its
  // neighbouring cells itself, in FP64.
  if (tid == 0) {
    TileHdr h;
    h.a0 = a0;
    h.a1 = a1;
    h.pad_ = 0;
    h.halo = -1;
    a.thdr[tix] = h;
  }
  for (int li = a0 + tid; li < a1; li += kListBlock) {
    const int64_t gi = g.atom_off + li;
    const double4 pi = P[li];
    const int tyi = (int)pi.w;
    double rl2[2];
    for (int b = 0; b < 2; ++b) {
      const double rc = sqrt(a.pp[2 * tyi + b].rc2) + a.skin;
      rl2[b] = rc * rc;
    }
    int c3[3];
    cell_of_pos<D>(bx, nc, pi, c3);
    uint32_t* L = a.nbl + g.nb_off + li;
    int na = 0, nb = 0;   // A neighbours from row 0 up, B neighbours from row max_nb - 1 down
    bool over = false;
    const int zlo = (D == 3) ? -1 : 0, zhi = (D == 3) ? 1 : 0;
    for (int dz = zlo; dz <= zhi; ++dz) {
      int cz2 = c3[2] + dz, iz = 0;
      if (D == 3) {
        if (cz2 < 0) { cz2 += nc[2]; iz = -1; }
        else if (cz2 >= nc[2]) { cz2 -= nc[2]; iz = 1; }
      }
      for (int dy = -1; dy <= 1; ++dy) {
        int cy2 = c3[1] + dy, iy = 0;
        if (cy2 < 0) { cy2 += nc[1]; iy = -1; }
        else if (cy2 >= nc[1]) { cy2 -= nc[1]; iy = 1; }
        for (int dx = -1; dx <= 1; ++dx) {
          int cx = c3[0] + dx, ix = 0;
          if (cx < 0) { cx += nc[0]; ix = -1; }
          else if (cx >= nc[0]) { cx -= nc[0]; ix = 1; }
          const int code = (ix + 1) + 3 * (iy + 1) + 9 * (iz + 1);
          double sh[3];
          box_shift(bx, ix, iy, iz, sh);
          const int c = (cz2 * nc[1] + cy2) * nc[0] + cx;
          for (int j = cs[c]; j < cs[c + 1]; ++j) {
            if (j == li && code == 13) continue;
            const double4 pj = P[j];
            const double ddx = (pj.x - pi.x) + sh[0];
            const double ddy = (pj.y - pi.y) + sh[1];
            const double ddz = (D == 3) ? (pj.z - pi.z) + sh[2] : 0.0;
            const double r2 = ddx * ddx + ddy * ddy + ddz * ddz;
            if (r2 < rl2[(int)pj.w]) {
              if (na + nb < a.max_nb) {
                const int row = (pj.w == 0.0) ? na : a.max_nb - 1 - nb;
                L[(int64_t)row * g.npad] = (uint32_t)j | ((uint32_t)code << kCodeShift);
              } else {
                over = true;
              }
              if (pj.w == 0.0) ++na; else ++nb;
            }
          }
        }
      }
    }
    if (over) atomicMax(a.overflow, na + nb);
    a.nbc[gi] = over ? 0 : na | (nb << 16);
    a.tord[gi] = li;
  }
}

}  // namespace

void launch_rebuild(const RebuildArgs& a, hipStream_t s, const int32_t* nc3_dev) {
  if (a.nreps <= 0 || a.nblk <= 0) return;
  hipLaunchKernelGGL(k_rb_grid, dim3(a.nreps), dim3(64), 0, s, a, nc3_dev);
  if (a.dim == 3) {
    hipLaunchKernelGGL(k_rb_bin<3>, dim3(a.nblk), dim3(kBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_rb_bin<2>, dim3(a.nblk), dim3(kBlock), 0, s, a);
  }
  hipLaunchKernelGGL(k_rb_scan, dim3(a.nreps), dim3(1024), 0, s, a);
  hipLaunchKernelGGL(k_rb_scatter, dim3(a.nblk), dim3(kBlock), 0, s, a);
  if (a.dim == 3) {
    hipLaunchKernelGGL(k_rb_perm<3>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_rb_back<3>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_rb_list<3>, dim3(a.ntile_blk), dim3(kListBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_rb_perm<2>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_rb_back<2>, dim3(a.nblk), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_rb_list<2>, dim3(a.ntile_blk), dim3(kListBlock), 0, s, a);
  }
}

}  // namespace aqs
