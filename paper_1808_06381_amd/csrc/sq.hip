// sq.hip -- structure factor of the blob centres (Results section, Eq.
// Sfactor) on gfx950: S(q) = |rho(q)|^2 / C, rho(q) = sum_c exp(-i q . R_c),
// for one configuration of each replica.
//
// Wavevectors.  A Lees-Edwards box with offset delta has its images at
// R + a Lx x + b (Ly y + delta x) + c Lz z; the wavevectors that give every
// image the same phase are
//   q = (2 pi mx / Lx, 2 pi my / Ly - 2 pi mx delta / (Lx Ly), 2 pi mz / Lz)
// for integer (mx, my, mz), so that q . R = 2 pi (mx sx + my sy + mz sz) in
// the sheared fractional coordinates sx = x / Lx - delta y / (Lx Ly),
// sy = y / Ly, sz = z / Lz.  The phase factorises,
//   exp(-i q . R_c) = A_c(mx) B_c(my),  A_c(mx) = exp(-2 pi i mx sx),
//   B_c(my) = exp(-2 pi i (my sy + mz sz)),
// so on an (mx, my) grid rho = sum_c A_c(mx) B_c(my) is a complex dense
// contraction over particles whose operands are generated on the fly: the
// work is FP64 arithmetic, not memory traffic (a particle's 24 bytes feed
// nx * ny complex products).
//
// With the mz phase on A, A_c(mx) = exp(-2 pi i (mx sx + mz sz)), B(-my) is the
// conjugate of B(my), so four real sums over the particles give a wavevector
// and its mirror:
//   P1 = sum Ar Br, P2 = sum Ai Bi, P3 = sum Ar Bi, P4 = sum Ai Br,
//   rho(mx, my) = (P1 - P2) + i (P3 + P4),  rho(mx, -my) = (P1 + P2) + i (P4 - P3),
// and my = 0 is the sum of A itself.
//
// Layout.  k_sq_partial: a block of sixteen waves takes one tile of 64 mx x 64
// values of my >= 1 and one chunk of one replica's rows.  Per group of 32
// particles the A and B tables go to LDS in runs of 8 entries (a sincospi for
// the run's first entry, complex multiplication by the particle's unit step
// for the others), then the contraction runs on the matrix cores: FP64 16 x 16
// x 4 MFMA, one 16 x 16 tile of (mx, my) and its four sums per wave, four
// particles per step.  Two table buffers: while all waves contract one group,
// the halves of the block take turns to build the next one's tables first, so
// that vector and matrix units work at the same time; a fixed wave prepares
// the particles (coordinates and unit steps) two groups ahead, their positions
// loaded three ahead.  The waves of the first my rows also sum A (my = 0).
// Bound by the FP64 matrix rate: at N = 1e6 and 64 x 129 wavevectors 0.64 ms
// (51 TFLOP/s of the 71 a large FP64 matrix product reaches; 1.42 ms with all
// 129 my values contracted, one table buffer and eight waves).
// k_sq_reduce: per replica and q, the chunks' partial sums in a fixed order,
// then |rho|^2 / C.  No floating-point atomics: the result is deterministic.
// Operand layout of v_mfma_f64_16x16x4f64 (checked on the device): lane l
// supplies A[l%16][l/16] and B[l/16][l%16] and receives D[4r + l/16][l%16]
// in accumulator register r.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "launch.h"
#include "sim_dev.h"

namespace {

constexpr int SQ_THREADS = 1024;
constexpr int SQ_TX = 64;        // mx per tile
constexpr int SQ_TY = 64;        // my >= 1 per block
constexpr int SQ_TYMAX = 160;    // my columns of a tile of partial sums at most
constexpr int SQ_P = 32;         // particles per LDS group (a multiple of 4)
constexpr int SQ_RUN = 8;        // table entries per sincospi (complex recurrence)
static_assert(SQ_TX == 16 * 4 && SQ_TY == 16 * 4 && SQ_THREADS == 16 * 64,
              "one 16 x 16 tile of (mx, my) per wave");
static_assert(SQ_P * (SQ_TX + SQ_TY) / SQ_RUN == SQ_THREADS / 2, "a half builds a group in one go");

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct SqChunk {
  int32_t rep;     // replica
  int32_t pad;
  int64_t row0;    // first row
  int64_t rows;    // rows of the chunk (all real particles)
};

}  // namespace

// my columns of a tile: the grid's, rounded up to 16, at most SQ_TYMAX
__host__ __device__ __forceinline__ int sq_tile_w(int ny) {
  const int w = (ny + 15) / 16 * 16;
  return w < SQ_TYMAX ? w : SQ_TYMAX;
}

// LDS of a block: two buffers of both tables (rows padded by one entry: the
// table writes, 16 particles of one run per 16 lanes, and the MFMA operand
// reads fall on distinct banks), and the prepared particles
struct SqLds {
  double2 A[2][SQ_P][SQ_TX + 1];
  double2 B[2][SQ_P][SQ_TY + 1];
  double2 stA[2][SQ_P], stB[2][SQ_P];  // unit steps exp(-2 pi i sx), exp(-2 pi i sy)
  double fs[2][3][SQ_P];               // sx, sy, mz sz
};

// partial[(chunk * ntile + tile) * SQ_TX * tile_w + o] = sum over the chunk's
// particles of A(mx) B(my), o = (mx - mx0) * tile_w + column, tile and column
// of my + my_max in tiles of tile_w columns (tiles_y per mx tile); complex as
// double2 (re, im).  blockIdx.x: mx tile * blocks_y + block of my values.
__global__ __launch_bounds__(SQ_THREADS) void k_sq_partial(DevPtrs d, const SqChunk* __restrict__ chunks,
                                                           int nx, int my_max, int mz, int blocks_y,
                                                           int tiles_y, int tile_w, int ntile,
                                                           double2* __restrict__ partial) {
  extern __shared__ __align__(16) char sq_lds[];
  SqLds& L = *reinterpret_cast<SqLds*>(sq_lds);
  const int by = blockIdx.x % blocks_y, ci = blockIdx.y;
  const SqChunk ch = chunks[ci];
  const RepDev& R = d.rep[ch.rep];
  const int xt = blockIdx.x / blocks_y, mx0 = xt * SQ_TX;
  const int my0 = 1 + by * SQ_TY;
  const double delta = le_offset(R, *d.step_d);
  const double ilx = 1.0 / R.L[0], ily = 1.0 / R.L[1], ilz = 1.0 / R.L[2];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave & 3, wn = wave >> 2;   // mx rows mx0 + 16 wm.., my values my0 + 16 wn..
  const int li = lane & 15, lk = lane >> 4;  // operand row / column, particle of the step
  // the waves of a SIMD (wave mod 4) share wm: with few my values every SIMD
  // keeps one busy wave
  const bool busy = mx0 + 16 * wm < nx && my0 + 16 * wn <= my_max;
  f64x4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
  // table building: a half's thread tb takes run tb / SQ_P of particle tb % SQ_P
  const int half = t / (SQ_THREADS / 2), tb = t % (SQ_THREADS / 2);
  const int bp = tb % SQ_P, brun = tb / SQ_P;
  const bool isA = brun < SQ_TX / SQ_RUN;
  const int k0 = (isA ? brun : brun - SQ_TX / SQ_RUN) * SQ_RUN;
  const bool used = isA ? mx0 + k0 < nx : my0 + k0 <= my_max;
  // my = 0: the waves of the first my rows also sum their A operands
  const bool sums = by == 0 && wn == 0 && mx0 + 16 * wm < nx;
  double s0r = 0.0, s0i = 0.0;
  const int groups = (int)((ch.rows + SQ_P - 1) / SQ_P);
  const bool prep = wave == 15 && lane < SQ_P;
  auto load_pos = [&](int g) {
    const int64_t i = (int64_t)g * SQ_P + lane;
    return prep && i < ch.rows ? d.pos[ch.row0 + i] : make_double4(0.0, 0.0, 0.0, 0.0);
  };
  auto particles = [&](int g, const double4& r) {
    if (!prep || g >= groups) return;
    const int q = g & 1;
    const double sx = r.x * ilx - delta * r.y * (ilx * ily);
    const double sy = r.y * ily;
    L.fs[q][0][lane] = sx;
    L.fs[q][1][lane] = sy;
    L.fs[q][2][lane] = (double)mz * (r.z * ilz);
    double ss, cs;
    sincospi(2.0 * sx, &ss, &cs);
    L.stA[q][lane] = make_double2(cs, -ss);
    sincospi(2.0 * sy, &ss, &cs);
    L.stB[q][lane] = make_double2(cs, -ss);
  };
  // tables of group g: A[p][mx - mx0], B[p][my - my0], in runs of SQ_RUN
  // consecutive entries: the first by sincospi, the others by complex
  // multiplication with the unit step (error <= 2 (SQ_RUN - 1) ulp, against
  // one sincospi per entry); rows past the chunk's particles are exact zeros
  auto build = [&](int g) {
    const int q = g & 1;
    double2* dst = isA ? &L.A[q][bp][k0] : &L.B[q][bp][k0];
    if ((int64_t)g * SQ_P + bp >= ch.rows || !used) {
#pragma unroll
      for (int j = 0; j < SQ_RUN; ++j) dst[j] = make_double2(0.0, 0.0);
      return;
    }
    double s0, c0;
    sincospi(isA ? 2.0 * ((double)(mx0 + k0) * L.fs[q][0][bp] + L.fs[q][2][bp])
                 : 2.0 * ((double)(my0 + k0) * L.fs[q][1][bp]),
             &s0, &c0);
    double zr = c0, zi = -s0;  // exp(-i phase); step u
    const double2 st = isA ? L.stA[q][bp] : L.stB[q][bp];
#pragma unroll
    for (int j = 0; j < SQ_RUN; ++j) {
      if (j > 0) {
        const double nr = fma(zr, st.x, -zi * st.y);
        const double ni = fma(zr, st.y, zi * st.x);
        zr = nr;
        zi = ni;
      }
      dst[j] = make_double2(zr, zi);
    }
  };
  particles(0, load_pos(0));
  particles(1, load_pos(1));
  double4 rnext = load_pos(2);
  __syncthreads();
  if (half == 0) build(0);
  __syncthreads();
  for (int g = 0; g < groups; ++g) {
    const int q = g & 1;
    // the step buffer of group g is free (its tables are built): group g + 2's
    particles(g + 2, rnext);
    rnext = load_pos(g + 3);
    if (half == ((g + 1) & 1) && g + 1 < groups) build(g + 1);
    if (sums) {
#pragma unroll
      for (int p0 = 0; p0 < SQ_P; p0 += 4) {
        const double2 a = L.A[q][p0 + lk][16 * wm + li];
        s0r += a.x;
        s0i += a.y;
      }
    }
    if (busy) {
#pragma unroll 2
      for (int p0 = 0; p0 < SQ_P; p0 += 4) {
        const double2 a = L.A[q][p0 + lk][16 * wm + li];
        const double2 b = L.B[q][p0 + lk][16 * wn + li];
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, acc[3], 0, 0, 0);
      }
    }
    __syncthreads();  // group g + 1's tables and group g + 2's steps are visible,
                      // group g's buffers free
  }
  // the partial sum of (mx0 + row, my)
  auto at = [&](int row, int my) -> double2& {
    const int col = my + my_max;
    return partial[((int64_t)ci * ntile + xt * tiles_y + col / tile_w) * ((int64_t)SQ_TX * tile_w) +
                   (int64_t)row * tile_w + col % tile_w];
  };
  if (busy) {
    const int my = my0 + 16 * wn + li;
    if (my <= my_max) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * wm + 4 * r + lk;
        at(row, my) = make_double2(acc[0][r] - acc[1][r], acc[2][r] + acc[3][r]);
        at(row, -my) = make_double2(acc[0][r] + acc[1][r], acc[3][r] - acc[2][r]);
      }
    }
  }
  if (sums) {  // over the four particle slots of a step
    s0r += __shfl_xor(s0r, 16, 64);
    s0i += __shfl_xor(s0i, 16, 64);
    s0r += __shfl_xor(s0r, 32, 64);
    s0i += __shfl_xor(s0i, 32, 64);
    if (lk == 0) at(16 * wm + li, 0) = make_double2(s0r, s0i);
  }
}

// out[(rep * nx + mx) * ny + (my + my_max)] = |sum of the replica's chunk
// partials|^2 / C: slice s of SQ_SLICES adds chunks s, s + SQ_SLICES, .. in
// order, then the slices in order (one thread per output walking all chunks
// of N = 1e6 took 73 us: 33 blocks of dependent loads)
constexpr int SQ_SLICES = 8;
constexpr int SQ_OUTS = 256 / SQ_SLICES;
__global__ __launch_bounds__(256) void k_sq_reduce(DevPtrs d, const int32_t* __restrict__ rep_chunk0,
                                                   int nrep, int nx, int my_max, int tiles_y,
                                                   int tile_w, int ntile,
                                                   const double2* __restrict__ partial,
                                                   double* __restrict__ out) {
  __shared__ double2 part[SQ_SLICES][SQ_OUTS];
  const int ny = 2 * my_max + 1;
  const int oi = threadIdx.x % SQ_OUTS, sl = threadIdx.x / SQ_OUTS;
  const int64_t o = (int64_t)blockIdx.x * SQ_OUTS + oi;
  const bool ok = o < (int64_t)nrep * nx * ny;
  const int rep = ok ? (int)(o / ((int64_t)nx * ny)) : 0;
  double re = 0.0, im = 0.0;
  if (ok) {
    const int q = (int)(o % ((int64_t)nx * ny));
    const int mx = q / ny, myi = q % ny;
    const int tile = (mx / SQ_TX) * tiles_y + myi / tile_w;
    const int off = (mx % SQ_TX) * tile_w + myi % tile_w;
#pragma unroll 4
    for (int c = rep_chunk0[rep] + sl; c < rep_chunk0[rep + 1]; c += SQ_SLICES) {
      const double2 v = partial[((int64_t)c * ntile + tile) * ((int64_t)SQ_TX * tile_w) + off];
      re += v.x;
      im += v.y;
    }
  }
  part[sl][oi] = make_double2(re, im);
  __syncthreads();
  if (sl != 0 || !ok) return;
  for (int k = 1; k < SQ_SLICES; ++k) {
    re += part[k][oi].x;
    im += part[k][oi].y;
  }
  const int n = d.rep[rep].n;
  out[o] = n > 0 ? (re * re + im * im) / (double)n : 0.0;
}

// ---------------------------------------------------------------------------
// host side: chunking and launches (device scratch from the caller)
// ---------------------------------------------------------------------------
namespace {
constexpr int64_t SQ_CHUNK = 4096;  // rows per block
}

int64_t sq_chunk_count(const std::vector<int64_t>& rep_rows) {
  int64_t c = 0;
  for (int64_t n : rep_rows) c += (n + SQ_CHUNK - 1) / SQ_CHUNK;
  return c;
}

int64_t sq_tile_count(int nx, int my_max) {
  const int ny = 2 * my_max + 1, w = sq_tile_w(ny);
  return (int64_t)((nx + SQ_TX - 1) / SQ_TX) * ((ny + w - 1) / w);
}

size_t sq_chunk_bytes() { return sizeof(SqChunk); }
size_t sq_partial_bytes(int64_t nchunk, int nx, int my_max) {
  return (size_t)nchunk * (size_t)sq_tile_count(nx, my_max) * SQ_TX *
         (size_t)sq_tile_w(2 * my_max + 1) * sizeof(double2);
}

// The chunk table of every replica built on the device (one thread walks the
// replicas: a handful of stores per chunk), so that a caller's scratch can
// be filled without a host table.
__global__ void k_sq_chunks(DevPtrs d, SqChunk* __restrict__ chunks, int32_t* __restrict__ rep_chunk0) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  int32_t c = 0;
  for (int r = 0; r < d.nrep; ++r) {
    rep_chunk0[r] = c;
    const RepDev& R = d.rep[r];
    for (int64_t a = 0; a < R.n; a += SQ_CHUNK)
      chunks[c++] = SqChunk{r, 0, R.row_off + a, min<int64_t>(SQ_CHUNK, (int64_t)R.n - a)};
  }
  rep_chunk0[d.nrep] = c;
}

namespace {
// blocks of my >= 1 values (one where there are none: my = 0 is its)
int sq_blocks_y(int my_max) { return std::max(1, (my_max + SQ_TY - 1) / SQ_TY); }
unsigned sq_blocks(int nx, int my_max) {
  return (unsigned)((nx + SQ_TX - 1) / SQ_TX * sq_blocks_y(my_max));
}
// the contraction's tables take more LDS than a kernel gets unasked
hipError_t allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k_sq_partial),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SqLds));
}
size_t up256(size_t b) { return (b + 255) / 256 * 256; }
}

// Bytes of caller scratch that launch_sq_scratch needs: chunk table, chunk
// offsets, partial sums (256-byte aligned pieces).
size_t sq_scratch_bytes(int64_t nchunk, int nrep, int nx, int my_max) {
  return up256(sizeof(SqChunk) * (size_t)std::max<int64_t>(nchunk, 1)) +
         up256(sizeof(int32_t) * (size_t)(nrep + 1)) +
         up256(sq_partial_bytes(std::max<int64_t>(nchunk, 1), nx, my_max));
}

// The same kernels as launch_sq with every table on the device: `scratch`
// (sq_scratch_bytes() bytes, 256-byte aligned) holds the chunk table, the
// chunk offsets and the partial sums, out_d receives replicas x nx x ny.
// Nothing is allocated and nothing is copied from the host; the launches
// are asynchronous on stream s.
hipError_t launch_sq_scratch(const DevPtrs& d, int64_t nchunk, int nx, int my_max, int mz,
                             void* scratch, double* out_d, hipStream_t s) {
  char* base = (char*)scratch;
  SqChunk* chunks = (SqChunk*)base;
  const size_t b_ch = up256(sizeof(SqChunk) * (size_t)std::max<int64_t>(nchunk, 1));
  int32_t* c0 = (int32_t*)(base + b_ch);
  const size_t b_c0 = up256(sizeof(int32_t) * (size_t)(d.nrep + 1));
  double2* partial = (double2*)(base + b_ch + b_c0);
  hipLaunchKernelGGL(k_sq_chunks, dim3(1), dim3(64), 0, s, d, chunks, c0);
  const int ny = 2 * my_max + 1;
  const int tile_w = sq_tile_w(ny);
  const int tiles_y = (ny + tile_w - 1) / tile_w;
  const int ntile = (int)sq_tile_count(nx, my_max);
  if (nchunk > 0) {
    const hipError_t e = allow_lds();
    if (e) return e;
    const int blocks_y = sq_blocks_y(my_max);
    hipLaunchKernelGGL(k_sq_partial, dim3(sq_blocks(nx, my_max), (unsigned)nchunk),
                       dim3(SQ_THREADS), sizeof(SqLds), s, d, (const SqChunk*)chunks, nx, my_max,
                       mz, blocks_y, tiles_y, tile_w, ntile, partial);
  }
  const int64_t nout = (int64_t)d.nrep * nx * ny;
  hipLaunchKernelGGL(k_sq_reduce, dim3((unsigned)((nout + SQ_OUTS - 1) / SQ_OUTS)), dim3(256), 0, s, d, c0,
                     d.nrep, nx, my_max, tiles_y, tile_w, ntile, partial, out_d);
  return hipGetLastError();
}

// rep_row0 / rep_rows: first row and real particles of each replica;
// chunks_d (sq_chunk_bytes() x count) and rep_chunk0_d (nrep + 1 int32)
// are device scratch, filled here from the host tables; ev0/ev1 (optional)
// bracket the contraction kernel's launch
hipError_t launch_sq(const DevPtrs& d, const std::vector<int64_t>& rep_row0,
                     const std::vector<int64_t>& rep_rows, int nx, int my_max, int mz,
                     void* chunks_d, int32_t* rep_chunk0_d, double2* partial_d, double* out_d,
                     hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  std::vector<SqChunk> ch;
  std::vector<int32_t> c0;
  for (size_t r = 0; r < rep_rows.size(); ++r) {
    c0.push_back((int32_t)ch.size());
    for (int64_t a = 0; a < rep_rows[r]; a += SQ_CHUNK)
      ch.push_back({(int32_t)r, 0, rep_row0[r] + a, std::min<int64_t>(SQ_CHUNK, rep_rows[r] - a)});
  }
  c0.push_back((int32_t)ch.size());
  hipError_t e;
  if (!ch.empty() &&
      (e = hipMemcpyAsync(chunks_d, ch.data(), ch.size() * sizeof(SqChunk), hipMemcpyHostToDevice, s)))
    return e;
  if ((e = hipMemcpyAsync(rep_chunk0_d, c0.data(), c0.size() * sizeof(int32_t),
                          hipMemcpyHostToDevice, s)))
    return e;
  const int ny = 2 * my_max + 1;
  const int tile_w = sq_tile_w(ny);
  const int tiles_y = (ny + tile_w - 1) / tile_w;
  const int ntile = (int)sq_tile_count(nx, my_max);
  if (!ch.empty()) {
    if ((e = allow_lds())) return e;
    const int blocks_y = sq_blocks_y(my_max);
    const dim3 g(sq_blocks(nx, my_max), (unsigned)ch.size()), b(SQ_THREADS);
    if (ev0 || ev1)
      hipExtLaunchKernelGGL(k_sq_partial, g, b, sizeof(SqLds), s, ev0, ev1, 0, d,
                            (const SqChunk*)chunks_d, nx, my_max, mz, blocks_y, tiles_y, tile_w,
                            ntile, partial_d);
    else
      hipLaunchKernelGGL(k_sq_partial, g, b, sizeof(SqLds), s, d, (const SqChunk*)chunks_d, nx,
                         my_max, mz, blocks_y, tiles_y, tile_w, ntile, partial_d);
  }
  const int64_t nout = (int64_t)rep_rows.size() * nx * ny;
  hipLaunchKernelGGL(k_sq_reduce, dim3((unsigned)((nout + SQ_OUTS - 1) / SQ_OUTS)), dim3(256), 0, s, d,
                     rep_chunk0_d, (int)rep_rows.size(), nx, my_max, tiles_y, tile_w, ntile,
                     partial_d, out_d);
  // host tables must outlive the asynchronous copies
  if ((e = hipStreamSynchronize(s))) return e;
  return hipGetLastError();
}
