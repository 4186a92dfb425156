// Fused D3Q19 pull stream + TRT+aB collide (Eqs. LBM_Stream, LBM_Collide, MRT
// with the rates of Eqs. TRTmatrix / TRTbulkmatrix, adaptive shell of Sec. 2.3.2).
//
// One thread per cell, one block per whole x-row group where rows are narrow,
// so that the +-1 x-shifted loads of a row stay inside the block and every
// source value is fetched from HBM once (wider rows are split into pieces; the
// x-shifted loads then fetch one shared line per piece twice).  The PDF slots of solid cells carry the boundary
// values of the particle links that stream out of them (written by the
// boundary kernel), so a fluid cell pulls 19 values without branching.  Wall
// layers are fixed, so the sweep knows from the cell's coordinates which
// values come from a wall: a cell next to a wall layer replaces them by the
// moving-wall bounce-back value f~_qbar(x) + 6 w_q (u_w . c_q) of Sec. 2.2
// (half-way walls), formed from its own post-collision values.  For z walls
// that is a branch uniform over a block (a block lies in one z plane).
// Solid and wall cells are updated like fluid cells: their results are never
// read (the boundary kernel rewrites every slot a fluid cell pulls from a
// solid cell), and letting every lane load and store keeps each wavefront's
// accesses whole cache lines (lanes that skipped their cell made partial-line
// writes, which cost a quarter of the bandwidth in a 16 % solid suspension).
//
// Collision in deviation variables g = f - w_q:
//   TRT in velocity space: g~_q = g_q - s+ (g+_q - e+_q) - s- (g-_q - e-_q),
//   which equals M^-1 S_TRT (m^eq - M f) because the moment rows of App. A are
//   each even or odd under q -> q-bar; plus, for rows 5 and 6 of M (kinetic
//   energy and its square), the rank-2 correction
//   w_q (s_b - s+) [M_4q (m4eq - m4)/N_4 + M_5q (m5eq - m5)/N_5]
//   with N_4 = 2/3, N_5 = 2 (M^-1 = W M^T diag(1/N)).  s_b is the TRT+B rate
//   in shell cells (TRT+aB), everywhere (TRT+B), or s+ (TRT, SRT).
#include "collide.hpp"

#include <algorithm>

namespace lbmdem {

// one domain: tiles of whole x-rows, or of row pieces on wide lattices (see
// sweep_tiles), gx x gy tiles per z plane, x fastest, handed to the XCDs in
// runs (see launch_sweep_t; 1: tile by tile, 0: one run each); the current
// buffer is read from the domain's step state.  The 19 rows of a (y, z) lie next to each other, so a
// block stores one contiguous run: 512^3 FP32 3.50-3.52 ms alone (5.85 TB/s)
// against 3.80 with a plane of N cells per direction.
constexpr int SWEEP_MAX_THREADS = 512;

// Non-temporal stores where every row starts on a 64-byte piece.  Elsewhere the
// line at the junction of two rows is written in two parts, which plain stores
// let the L2 join: 75 x 61 x 101 FP32 22 -> 17 us, 429 x 151 x 100 277 -> 204,
// 150 x 130 x 140 FP64 198 -> 190, a batch of 16 requests 1.59 -> 1.35 ms (aligned
// rows lose: 384^3 1.54 -> 1.64 ms, 128x128x256 FP64 220 -> 243 us, 200^3 FP64
// 453 -> 482 us).  With a body force the same: aligned rows 128x128x256 FP64 246 ->
// 220 us, 384^3 FP32 1.64 -> 1.50 ms with non-temporal stores.
__host__ __device__ inline bool nt_stores(int nx, int size) { return nx * size % 64 == 0; }

template <typename T, bool FORCED, bool NTLOAD, bool NTSTORE>
__global__ __launch_bounds__(SWEEP_MAX_THREADS) void k_sweep(DevDomain d, int gx, int gy, int run) {
  using C = typename Store<T>::C;
  if (!step_live(d.ctl)) return;
  const int t = run == 1 ? (int)blockIdx.x : (run ? xcd_run_tile((int)blockIdx.x, run) : xcd_tile((int)blockIdx.x, (int)gridDim.x));
  const int bx = t % gx, r = t / gx, by = r % gy, z = r / gy;
  if (z >= d.nz) return;
  const int cur = d.ctl->cur;
  const int x = bx * blockDim.x + threadIdx.x;
  const int y = by * blockDim.y + threadIdx.y;
  if (x >= d.nx || y >= d.ny) return;
  // (selects, not an index: a run-time index into the by-value argument would
  // place the whole descriptor in scratch memory)
  const T* src = (const T*)(cur ? d.pdf[1] : d.pdf[0]);
  T* dst = (T*)(cur ? d.pdf[0] : d.pdf[1]);
  sweep_cell<T, FORCED, NTLOAD, NTSTORE>(d, src, dst, x, y, z, (C)d.s_plus, (C)d.s_minus,
                        (C)(d.s_bulk_shell - d.s_plus), (C)(d.s_bulk_other - d.s_plus));
}

// many domains in one launch: block b belongs to the domain k with
// start[k] <= b < start[k+1] and covers one tile of it.  Tiles are whole rows
// (or row pieces) as in the single sweep: tiles of 256 consecutive cells, cut
// anywhere in a row, share the lines at both cuts of all 19 rows with another
// block (16 requests of 48-192 cells a side, 31.8 M cells, FP32: 2.10 ms;
// 1.52 ms with a plane of N cells per direction; whole rows 1.35 ms; more rows
// per block 1.46 ms at 512 cells, 1.69 at 1024).  The code of forced cells is
// in a kernel of its own: beside it the unforced one takes 86 VGPRs instead of
// 67 (steps of 8 domains: 150 x 130 x 140 FP32 732 -> 697 us, 130^3 626 -> 574,
// 128^3 FP16 317 -> 303; 75 x 61 x 101 167 -> 172).  Forced cells are stored
// plainly: 8 x 128^3 FP32 454 us a step, 463 with non-temporal stores.
template <typename T, bool FORCED>
__global__ __launch_bounds__(SWEEP_MAX_THREADS) void k_sweep_batch(const DevDomain* __restrict__ tab,
                                                     const int* __restrict__ start, int ndom) {
  using C = typename Store<T>::C;
  const int k = batch_domain(start, ndom, (int)blockIdx.x);
  const DevDomain& d = tab[k];
  if (!step_live(d.ctl)) return;
  const int t = (int)blockIdx.x - start[k];
  const int bx = t % d.sw_gx, r = t / d.sw_gx, by = r % d.sw_gy, z = r / d.sw_gy;
  const int ty = (int)threadIdx.x / d.sw_bx;
  const int x = bx * d.sw_bx + (int)threadIdx.x - ty * d.sw_bx, y = by * d.sw_by + ty;
  if (ty >= d.sw_by || x >= d.nx || y >= d.ny) return;
  const int cur = d.ctl->cur;
  const T* src = (const T*)d.pdf[cur];
  T* dst = (T*)d.pdf[cur ^ 1];
  const C sp = (C)d.s_plus, sm = (C)d.s_minus, dbs = (C)(d.s_bulk_shell - d.s_plus), dbo = (C)(d.s_bulk_other - d.s_plus);
  if (FORCED && d.forced)  // uniform over the block (one domain)
    sweep_cell<T, true, false, false>(d, src, dst, x, y, z, sp, sm, dbs, dbo);
  else if (nt_stores(d.nx, (int)sizeof(T)))
    sweep_cell<T, false, false, true>(d, src, dst, x, y, z, sp, sm, dbs, dbo);
  else
    sweep_cell<T, false, false, false>(d, src, dst, x, y, z, sp, sm, dbs, dbo);
}

// Tile shape.  Bounded by HBM bandwidth; what the shape changes is how many
// tiles share cache lines and which of its L2's channels an XCD uses.  Rows of
// whole 64-byte pieces: whole rows (256 / nx of them) up to 256 cells, 512 at
// FP16, 128 at FP64; wider ones in pieces (row_piece).  Other rows share the
// line at each junction of their 19 rows, so they stay whole up to 512 cells, 256
// at FP64 (429 x 151 x 100: FP32 204 us against 222 in 215s; FP64 428 us in 215s
// against 474 whole), wider ones in equal pieces.  In a batch, whose blocks all
// have the threads of the largest tile, the wide FP16 rows of whole pieces stay
// in up to 256s (8 x 384 x 64 x 64: 248 us a step against 285 whole), the other
// rows whole (8 x 300 x 100 x 90 FP32 675 us a step against 792 in 150s).
//
// Pieces of rows of whole 64-byte pieces: whole 128-byte lines, and either an odd
// number of them or 1 KB each.  Tiles go to the eight XCDs one by one, so with an
// even number an XCD keeps getting the same columns, and with short pieces only a
// few channels of its L2.  GB/s, sweep alone: FP32 768 x 256 x 256 in six 128s 5,220, in
// three 256s 5,640; 1024 x 256 x 256 in eight 128s 5,450, in five 224s 5,830, in four
// 256s 5,940; 512 x 128 x 128 in four 128s 5,580, in three 192s 5,870, in two 256s 5,870; FP16
// 1024 x 256 x 256 in eight 128s 5,010, in three 384s 6,000, in two 512s 5,920; FP64 512 x 128
// x 128 in four 128s 5,790, in three 176s 5,760.  Pieces that end inside a line cost most:
// equal parts of 182 to 253 cells of rows of 544 to 992 ran at 3,700 to 4,300, three or
// five pieces of whole lines run at 5,550 to 5,940 (FP64 4,200 to 4,560 and 5,170 to 5,800,
// FP16 3,760 to 4,080 and 5,270 to 5,550).  A row that an odd number of 128s, 64s, 160s or
// 96s fills exactly is cut so (384^3 FP32 128 x 2, 320^3 64 x 4, 480 x 160 x 82 160 x 1: 1 %
// above whole rows).
static int row_piece(int nx, int size, int widest) {
  const int line = 128 / size, cand[6] = {128, 64, 160, 96, 256, 512}, least = (nx + widest - 1) / widest;
  for (int c : cand)
    if (nx % c == 0 && c % line == 0 && c <= widest && (nx / c % 2 == 1 || c * size >= 1024)) return c;
  if (least == 1) return nx;
  auto piece = [&](int n) { return ((nx + n - 1) / n + line - 1) / line * line; };
  for (int n = least | 1; n < least + 16; n += 2)
    if (piece(n) <= widest && (nx + piece(n) - 1) / piece(n) % 2 == 1) return piece(n);
  return piece(least);
}

void sweep_tiles(int nx, int ny, int storage, bool batch, int* bx, int* by, int* gx, int* gy) {
  const int size = storage == 0 ? 8 : (storage == 1 ? 4 : 2);
  const bool lines = nt_stores(nx, size);
  const int whole = lines ? (storage == 2 ? (batch ? 256 : 512) : (storage == 1 ? 256 : 128)) : (storage == 0 ? 256 : 512);
  const int widest = std::max(whole, 256), n = (nx + widest - 1) / widest;
  *bx = nx <= whole ? nx : (lines ? row_piece(nx, size, widest) : (nx + n - 1) / n);
  *by = *bx < 256 ? 256 / *bx : 1;
  *gx = (nx + *bx - 1) / *bx;
  *gy = (ny + *by - 1) / *by;
}

// LDS that a sweep block of so many threads asks for (and does not use) so that
// at most `waves` wavefronts of the sweep are resident on a CU.  The sweep is
// bound by bandwidth and needs no more; with eight of its waves on every SIMD
// (60 VGPRs each at FP32) no registers are left for a DEM wave (163-250 VGPRs)
// beside it, and the DEM chain waits for waves of the sweep to end together:
// 24,000 spheres beside the 512^3 FP32 sweep, sub-cycle 213 -> 61 us, first
// positions 1,000 -> 21 us, sweep 3.55 -> 3.52 ms; one sphere beside the
// 128x128x256 sweep 111 -> 46 us (FP64 148 -> 46).  20 waves per CU at FP32 and
// FP64; at FP16 (51 VGPRs) 24, where 20 slow the sweep (1.98 against 1.85 ms).
// The batch's sweep, with few DEM blocks beside it, is faster without (1.36 ms;
// 1.37 at 20, 1.46 at 16).
static unsigned residency_lds(int threads, int waves) {
  constexpr unsigned LDS_CU = 160u * 1024u;
  const int per_block = (threads + 63) / 64;
  const unsigned blocks = (unsigned)std::max(2, waves / per_block);
  return (LDS_CU / (blocks + 1) + 1024u) & ~511u;
}

template <typename T>
static void launch_sweep_t(const DevDomain& d, bool beside, hipStream_t s) {
  int bx, by, gx, gy;
  sweep_tiles(d.nx, d.ny, d.storage, false, &bx, &by, &gx, &gy);
  const dim3 block((unsigned)bx, (unsigned)by);
  const bool lines = nt_stores(d.nx, (int)sizeof(T));
  // Tile order: tile by tile over the XCDs, x fastest, except
  // - pieces of rows that share lines: one contiguous run of tiles per XCD (1000 x
  //   150 x 80 FP32 392 against 408 us);
  // - FP32 and FP16 buffers of more than 2 GB: runs of 128 tiles, so that an XCD
  //   touches fewer pages at a time, unless the row has five or more pieces of an odd
  //   number.  GB/s tile by tile / in runs of 128 / in one run: FP32 512^3 (10 GB, two
  //   256s) 5,640 / 5,880 / 5,830, 384^3 (4.3, three 128s) 5,680 / 5,840 / 5,670, 256 x 512 x
  //   512 (5.1) 5,580 / 5,820 / 5,740, 128 x 512 x 1024 (5.1) 5,530 / 5,780 / 5,690, FP16 512^3
  //   (5.1) 5,720 / 5,880 / 5,740; 320^3 FP32 (2.5, five 64s) 5,940 / 5,840, 640 x 512 x 512
  //   FP16 (6.4, five 128s) 6,100 / 5,780.  Smaller: 256^3 FP32 (1.3) 5,780 / 5,770 / 5,570,
  //   128x128x256 (0.3) 5,795 / 5,640 / 5,430.  FP64 gains and loses (384^3 5,380 / 5,490 /
  //   5,500, 256 x 384 x 384 5,590 / 5,500 / 5,460).
  const bool runs = sizeof(T) < 8 && (double)Q * (double)d.N * sizeof(T) > 2e9 && (gx < 5 || gx % 2 == 0);
  const int run = gx > 1 && !lines ? 0 : (runs ? 128 : 1);
  const int tiles = gx * gy * d.nz;
  const dim3 grid(run == 1 ? tiles : (run ? xcd_run_grid(tiles, run) : xcd_grid(tiles)));
  // Each value is read once, but a line that two waves share is read twice and
  // should still be cached then: plain loads (384^3 FP32 1.49 against 1.55 ms,
  // 320^3 826 against 933 us, 128x128x256 110 against 113 us).  At FP64 a wave
  // covers four whole lines and non-temporal loads win (128x128x256 217
  // against 223 us).
  constexpr bool nt = sizeof(T) == 8;
  const unsigned lds = beside ? residency_lds(bx * by, sizeof(T) == 2 ? 24 : 20) : 0u;
  if (d.forced && lines)
    hipLaunchKernelGGL((k_sweep<T, true, nt, true>), grid, block, lds, s, d, gx, gy, run);
  else if (d.forced)
    hipLaunchKernelGGL((k_sweep<T, true, nt, false>), grid, block, lds, s, d, gx, gy, run);
  else if (lines)
    hipLaunchKernelGGL((k_sweep<T, false, nt, true>), grid, block, lds, s, d, gx, gy, run);
  else
    hipLaunchKernelGGL((k_sweep<T, false, nt, false>), grid, block, lds, s, d, gx, gy, run);
}

void launch_sweep(const DevDomain& d, bool beside, hipStream_t s) {
  if (d.storage == 0)
    launch_sweep_t<double>(d, beside, s);
  else if (d.storage == 1)
    launch_sweep_t<float>(d, beside, s);
  else
    launch_sweep_t<__half>(d, beside, s);
}

template <typename T>
static void launch_sweep_batch_t(const BatchTables& b, hipStream_t s) {
  const dim3 grid(b.sweep_blocks), block(b.sweep_threads);
  if (b.forced)
    hipLaunchKernelGGL((k_sweep_batch<T, true>), grid, block, 0, s, b.tab, b.sweep_start, b.ndom);
  else
    hipLaunchKernelGGL((k_sweep_batch<T, false>), grid, block, 0, s, b.tab, b.sweep_start, b.ndom);
}

void launch_sweep_batch(const BatchTables& b, hipStream_t s) {
  if (b.sweep_blocks <= 0) return;
  if (b.storage == 0)
    launch_sweep_batch_t<double>(b, s);
  else if (b.storage == 1)
    launch_sweep_batch_t<float>(b, s);
  else
    launch_sweep_batch_t<__half>(b, s);
}

}  // namespace lbmdem
