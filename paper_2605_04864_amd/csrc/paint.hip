// Catalog sums, normalisations and FKP mass assignment (CIC / TSC, interlacing).
//
// Painting: particles are counting-sorted by 16^3-node tile (two LDS-staged
// steps: by bucket of tiles, then by tile; for the FP32 painter on meshes of
// 256^3 and more the records are 8-byte tile-relative ones from the first step
// on, with a 16-bit tile index beside them up to 2^16 tiles), each tile's
// particles are
// accumulated into a 19^3-node LDS block (the tile plus the stencil halo) with
// LDS atomics, blocks are written out without atomics, and a fold pass sums
// the <= 8 blocks covering every node while forming delta = n_g - alpha n_r and
// N = n_g(w^2) + alpha^2 n_r(w^2).
#include "fft.h"
#include "paint.h"

namespace cnpc {

constexpr int TILE = 16;
constexpr int BW = TILE + 3;           // block width: nodes c-1 .. c+2 around tile
constexpr int BVOL = BW * BW * BW;     // 6859
constexpr int BSTRIDE = 6880;          // elements per (tile, phase) block: BVOL rounded to 32

// Layout of a block (LDS accumulator and memory).  Local node l = 0..18 along
// an axis is node 16 t - 1 + l of the mesh: l = 1..16 are the tile's own
// nodes, l = 17..18 nodes 0..1 of the upper neighbour, l = 0 node 15 of the
// lower one.  Rows (lx, ly) of 19 nodes are stored in row-major order, and
// within a row node lz sits at (lz + 18) mod 19: the 16 own nodes first, then
// the two of the upper neighbour, then the one of the lower neighbour.  So a
// fold reads every row as one run of 16 own values and short runs for the z
// neighbours, and the stencil addresses of a particle stay affine except for
// a node l = 0, which moves to the end of its row.
constexpr int SORT_BLOCK = 1024;
constexpr int SORT_PER_THREAD = 64;    // particles per thread per sort workgroup
constexpr int LDS_TILES_MAX = 8192;    // LDS-aggregated sort up to this many tiles

// ------------------------------------------------------------ tile keys --
struct TileGeom {
  int shift;  // 32 - log2(n): node index = p >> shift
  int nt;     // tiles per side
  int ls;     // log2(S)
  int lnb;    // log2(buckets per side)
};

template <int RS>
struct Rec {
  uint32_t v[RS];
};

// Tile-sorted record of the FP32 painter (unweighted catalogs, meshes of 256^3
// and more): the 21 bits of each coordinate below the tile index, i.e. the 4
// node bits inside the 16-node tile and the top 17 fraction bits, in 8 bytes
// (x | y << 21 | z << 42).  Positions keep a 2^-17 cell grid, finer than FP32
// coordinates of a 256-cell box resolve; needs shift >= 17 (meshes up to 2^15
// per side).  The grid's jitter scales with the cell size, so coarser meshes,
// whose binned k reach closer to their Nyquist wavenumber, keep full records.
__host__ __device__ constexpr bool packs_records(bool f32, int rs, int shift) {
  return f32 && rs == 3 && shift <= 24;
}
__device__ __forceinline__ uint64_t pack_rec(const Rec<3>& r, int shift) {
  const uint32_t m = shift + 4 >= 32 ? 0xffffffffu : ((1u << (shift + 4)) - 1u);
  const int down = shift - 17;
  return (uint64_t)((r.v[0] & m) >> down) | ((uint64_t)((r.v[1] & m) >> down) << 21) |
         ((uint64_t)((r.v[2] & m) >> down) << 42);
}

// a tile-sorted record out: in full, or packed (pack_rec) for the FP32 painter
template <int RS>
__device__ __forceinline__ void put_rec(Rec<RS>* out, uint32_t o, const Rec<RS>& r, bool pack, int shift) {
  if constexpr (RS == 3) {
    if (pack) {
      reinterpret_cast<uint64_t*>(out)[o] = pack_rec(r, shift);
      return;
    }
  }
  out[o] = r;
}

// catalog positions read once by the sums pass: non-temporal loads
__device__ __forceinline__ uint32_t ld_stream(const uint32_t* p) { return __builtin_nontemporal_load(p); }

__device__ __forceinline__ int key_of(int tx, int ty, int tz, const TileGeom& g) {
  const int m = (1 << g.ls) - 1;
  const int b = ((((tx >> g.ls) << g.lnb) | (ty >> g.ls)) << g.lnb) | (tz >> g.ls);
  const int l = ((((tx & m) << g.ls) | (ty & m)) << g.ls) | (tz & m);
  return (b << (3 * g.ls)) | l;
}

__device__ __forceinline__ int tile_key(uint32_t px, uint32_t py, uint32_t pz, const TileGeom& g) {
  return key_of((int)(px >> g.shift) >> 4, (int)(py >> g.shift) >> 4, (int)(pz >> g.shift) >> 4, g);
}

struct CountArgs {
  TileGeom g;
  int ntiles;
  uint32_t* count;  // nullptr: sums only
};

// ------------------------------------------------------------ catalog sums --
// v shifted by one DPP control word (zero where it takes from no lane)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// sum over the wavefront, in every lane.  Row shifts and row broadcasts on the
// VALU: as 64-bit lane permutes through the LDS pipe, the 21 sums of a
// 1024-thread workgroup took 13 us at the end of every sums and bucket pass.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8: lane 15 of each row of 16 holds the row's sum
  v += dpp_f64<0x112, 0xf>(v);
  v += dpp_f64<0x114, 0xf>(v);
  v += dpp_f64<0x118, 0xf>(v);
  v += dpp_f64<0x142, 0xa>(v);  // row_bcast:15 into rows 1, 3
  v += dpp_f64<0x143, 0xc>(v);  // row_bcast:31 into rows 2, 3
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, 63);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// columns of the catalog sums that LMAX leaves non-zero (the imaginary part of
// every m = 0 sum is zero too)
__host__ __device__ constexpr int sums_used(int lmax) { return lmax >= 4 ? CNPC_SUMS_LEN : lmax >= 2 ? 11 : 4; }

constexpr int SUMS_THREADS = 1024;
constexpr int SUMS_BLOCKS = 256;

// adds the catalog sums of one particle (weight wi) to acc
template <int LMAX>
__device__ __forceinline__ void sums_add(double* acc, uint32_t px, uint32_t py, uint32_t pz, double wi,
                                       double scale, const SumsArgs& a) {
  const double w2 = wi * wi, w3 = w2 * wi;
  acc[0] += wi;
  acc[1] += w2;
  acc[2] += w3;
  int q = 3;
  // (l, m) order: (0,0), (2,0..2), (4,0..4); accumulate w^3 conj(y_l^m)
  acc[q++] += w3;  // y_0^0 = 1
  acc[q++] += 0.0;
  if constexpr (LMAX < 2) return;
  if (a.global_los) {
    double re[5], im[5];
    racah_ylm<double>(2, a.los[0], a.los[1], a.los[2], re, im);
    for (int m = 0; m <= 2; ++m) { acc[q++] += w3 * re[m]; acc[q++] -= w3 * im[m]; }
    if constexpr (LMAX < 4) return;
    racah_ylm<double>(4, a.los[0], a.los[1], a.los[2], re, im);
    for (int m = 0; m <= 4; ++m) { acc[q++] += w3 * re[m]; acc[q++] -= w3 * im[m]; }
  } else {
    // solid harmonics: y_l^m(r / R) = Q_lm(r_z, R^2) (r_x + i r_y)^m / R^l,
    // the Q_lm of solid_coef written out for l = 2, 4
    const double rx = (double)px * scale - a.obs[0];
    const double ry = (double)py * scale - a.obs[1];
    const double rz = (double)pz * scale - a.obs[2];
    const double z2 = rz * rz;
    const double r2 = rx * rx + ry * ry + z2;
    const double i2 = 1.0 / r2;
    const double c2 = w3 * i2, c4 = c2 * i2;
    const double s2r = rx * rx - ry * ry, s2i = 2.0 * rx * ry;
    const double s3r = s2r * rx - s2i * ry, s3i = s2r * ry + s2i * rx;
    const double s4r = s2r * s2r - s2i * s2i, s4i = 2.0 * s2r * s2i;
    const double q20 = c2 * (1.5 * z2 - 0.5 * r2);
    const double q21 = c2 * -1.22474487139158904910 * rz;
    const double q22 = c2 * 0.61237243569579452455;
    acc[5] += q20;
    acc[7] += q21 * rx; acc[8] -= q21 * ry;
    acc[9] += q22 * s2r; acc[10] -= q22 * s2i;
    if constexpr (LMAX < 4) return;
    const double q40 = c4 * ((4.375 * z2 - 3.75 * r2) * z2 + 0.375 * r2 * r2);
    const double q41 = c4 * rz * (-3.91311896062463196870 * z2 + 1.67705098312484227230 * r2);
    const double q42 = c4 * (2.76699295264733191550 * z2 - 0.39528470752104741650 * r2);
    const double q43 = c4 * -1.47901994577490951707 * rz;
    const double q44 = c4 * 0.52291251658379721749;
    acc[11] += q40;
    acc[13] += q41 * rx; acc[14] -= q41 * ry;
    acc[15] += q42 * s2r; acc[16] -= q42 * s2i;
    acc[17] += q43 * s3r; acc[18] -= q43 * s3i;
    acc[19] += q44 * s4r; acc[20] -= q44 * s4i;
  }
}

// Catalog sums of one workgroup, block `blk` of `nblk` (LMAX: Y_lm sums for
// l <= LMAX, 0, 2 or 4; the others stay zero; its particles are those of every
// nblk-th run of SUMS_THREADS, so that the workgroups read one stretch of the catalog
// at a time: with a range of its own for each, 3e8 particles took 1274 us, 1183
// here) into partial[blk], and the tile
// histogram of its particles: with `hist` stored there (at most 64 tiles), else
// added to ca.count.
constexpr int SMALL_TILES = 64;  // tiles of a mesh of one bucket, at most
template <int LMAX>
__device__ __forceinline__ void catalog_sums_block(const uint32_t* __restrict__ pos, const float* __restrict__ w,
                                                   int64_t n, const SumsArgs& a, double* __restrict__ partial,
                                                   const CountArgs& ca, uint32_t* __restrict__ hist, int blk, int nblk) {
  extern __shared__ uint32_t lcount[];
  const bool count = ca.count != nullptr || hist != nullptr;
  const bool lds = count && ca.ntiles <= LDS_TILES_MAX;
  if (lds) {
    for (int t = threadIdx.x; t < ca.ntiles; t += blockDim.x) lcount[t] = 0;
    __syncthreads();
  }
  double acc[CNPC_SUMS_LEN];
#pragma unroll
  for (int q = 0; q < CNPC_SUMS_LEN; ++q) acc[q] = 0.0;
  const double scale = a.boxsize / 4294967296.0;
  // U particles per thread and trip: all their loads are issued before any of
  // them is used (fewer for the larger register sets of l > 0)
  constexpr int U = LMAX == 0 ? 4 : (LMAX == 2 ? 2 : 1);
  const int64_t stride = (int64_t)nblk * SUMS_THREADS;
  for (int64_t i0 = (int64_t)blk * SUMS_THREADS + threadIdx.x; i0 < n; i0 += U * stride) {
    uint32_t px[U], py[U], pz[U];
    float wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      px[u] = py[u] = pz[u] = 0u;
      wv[u] = 1.0f;
      if (i < n) {
        px[u] = ld_stream(pos + i);
        py[u] = ld_stream(pos + n + i);
        pz[u] = ld_stream(pos + 2 * n + i);
        if (w) wv[u] = w[i];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * stride >= n) break;
      if (count) {
        const int t = tile_key(px[u], py[u], pz[u], ca.g);
        if (lds) atomicAdd(&lcount[t], 1u);
        else atomicAdd(&ca.count[t], 1u);
      }
      sums_add<LMAX>(acc, px[u], py[u], pz[u], (double)wv[u], scale, a);
    }
  }
  __shared__ double red[SUMS_THREADS / 64][CNPC_SUMS_LEN];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < CNPC_SUMS_LEN; ++q) {
    const double v = q < sums_used(LMAX) ? wave_sum(acc[q]) : 0.0;
    if (lane == 0) red[wv][q] = v;
  }
  __syncthreads();
  if (threadIdx.x < CNPC_SUMS_LEN) {
    double v = 0.0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) v += red[k][threadIdx.x];
    partial[(int64_t)blk * CNPC_SUMS_LEN + threadIdx.x] = v;
  }
  if (lds) {
    for (int t = threadIdx.x; t < ca.ntiles; t += blockDim.x) {
      const uint32_t c = lcount[t];
      if (hist) hist[(int64_t)blk * SMALL_TILES + t] = c;
      else if (c) atomicAdd(&ca.count[t], c);
    }
  }
}

template <int LMAX>
__global__ void __launch_bounds__(SUMS_THREADS) k_catalog_sums(const uint32_t* __restrict__ pos,
                                                      const float* __restrict__ w, int64_t n,
                                                      SumsArgs a, double* __restrict__ partial,
                                                      CountArgs ca) {
  catalog_sums_block<LMAX>(pos, w, n, a, partial, ca, nullptr, blockIdx.x, gridDim.x);
}

// Both catalogs of a painting, for the kernels that take them in one launch on
// meshes of one tile bucket (blockIdx.y: galaxies, randoms).
struct SmallCat {
  const uint32_t* pos;
  const float* w;
  int64_t n;
  int nblk;           // workgroups of its sums
  double* partial;    // [nblk][CNPC_SUMS_LEN]
  uint32_t* hist;     // [nblk][SMALL_TILES] tile histograms, then the workgroups' slots
  uint32_t *count, *start;  // [ntiles]
  void* rec;          // tile-sorted records
  double* sums;
};
struct SmallPair {
  SmallCat c[2];
};

template <int LMAX>
__global__ void __launch_bounds__(SUMS_THREADS) k_catalog_sums2(SmallPair sp, SumsArgs a, TileGeom g, int ntiles) {
  const SmallCat c = sp.c[blockIdx.y];
  if ((int)blockIdx.x >= c.nblk) return;
  CountArgs ca;
  ca.g = g;
  ca.ntiles = ntiles;
  ca.count = nullptr;
  catalog_sums_block<LMAX>(c.pos, c.w, c.n, a, c.partial, ca, c.hist, blockIdx.x, c.nblk);
}

__global__ void __launch_bounds__(64) k_reduce_partials(const double* __restrict__ partial, int nblocks,
                                                        double* __restrict__ out) {
  // block q sums column q over the partials in a fixed order (deterministic)
  const int q = blockIdx.x;
  double v = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += 64) v += partial[(int64_t)b * CNPC_SUMS_LEN + q];
  v = wave_sum(v);
  if (threadIdx.x == 0) out[q] = v;
}

__device__ __forceinline__ void form_norms(const double* gs, const double* rs, int64_t ngal, double boxsize,
                                           double* __restrict__ nm) {
  const double alpha = gs[0] / rs[0];
  const double nbar = (double)ngal / (boxsize * boxsize * boxsize);
  const double I22 = alpha * nbar * rs[1];
  const double I33 = alpha * nbar * nbar * rs[2];
  nm[CNPC_NORM_ALPHA] = alpha;
  nm[CNPC_NORM_NBAR] = nbar;
  nm[CNPC_NORM_I22] = I22;
  nm[CNPC_NORM_I33] = I33;
  nm[CNPC_NORM_N0] = (gs[1] + alpha * alpha * rs[1]) / I22;
  nm[CNPC_NORM_SBAR] = gs[2] - alpha * alpha * alpha * rs[2];
  const double a3 = alpha * alpha * alpha;
  for (int q = 0; q < 2 * CNPC_NYLM_SUMS; ++q) nm[CNPC_NORM_SBARLM + q] = gs[3 + q] - a3 * rs[3 + q];
}

__global__ void k_norms(const double* __restrict__ gs, const double* __restrict__ rs, int64_t ngal,
                        double boxsize, double* __restrict__ nm) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  form_norms(gs, rs, ngal, boxsize, nm);
}

// The steps between the sums and the sort of a mesh of one tile bucket, one
// launch: workgroups 0, 1 add the tile histograms of a catalog's sums workgroups,
// scan them (count, start) and leave in hist[b][t] where workgroup b's particles of
// tile t go; workgroup 2 forms the catalog sums of both (k_reduce_partials' order)
// and, with nm, the norms.
__global__ void __launch_bounds__(1024) k_small_scan(SmallPair sp, int ntiles, int64_t ngal, double boxsize,
                                                     double* __restrict__ nm) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (blockIdx.x < 2) {
    const SmallCat c = sp.c[blockIdx.x];
    __shared__ uint32_t part[16][SMALL_TILES];
    constexpr int PB = SUMS_BLOCKS / 16;  // sums workgroups per wavefront: PB wv .. PB wv + PB - 1
    uint32_t h[PB], v = 0;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      const int b = PB * wv + k;
      h[k] = b < c.nblk && lane < ntiles ? c.hist[(int64_t)b * SMALL_TILES + lane] : 0u;
      v += h[k];
    }
    part[wv][lane] = v;
    __syncthreads();
    uint32_t cnt = 0, mine = 0;  // all wavefronts, the ones before this
    for (int k = 0; k < 16; ++k) {
      const uint32_t u = part[k][lane];
      if (k < wv) mine += u;
      cnt += u;
    }
    uint32_t run = cnt;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t u = __shfl_up(run, off, 64);
      if (lane >= off) run += u;
    }
    if (lane >= ntiles) return;
    if (wv == 0) {
      c.count[lane] = cnt;
      c.start[lane] = run - cnt;
    }
    uint32_t base = run - cnt + mine;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      const int b = PB * wv + k;
      if (b < c.nblk) c.hist[(int64_t)b * SMALL_TILES + lane] = base;
      base += h[k];
    }
    return;
  }
  __shared__ double sums[2][CNPC_SUMS_LEN];
  for (int q = wv; q < 2 * CNPC_SUMS_LEN; q += 16) {
    const int k = q >= CNPC_SUMS_LEN ? 1 : 0, col = q - k * CNPC_SUMS_LEN;
    double v = 0.0;
    for (int b = lane; b < sp.c[k].nblk; b += 64) v += sp.c[k].partial[(int64_t)b * CNPC_SUMS_LEN + col];
    v = wave_sum(v);
    if (lane == 0) {
      sums[k][col] = v;
      sp.c[k].sums[col] = v;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && nm) form_norms(sums[0], sums[1], ngal, boxsize, nm);
}

// ------------------------------------------------------------------- sort --
// Tiles are numbered bucket-major: a bucket is a cube of S^3 tiles (S = min(4,
// nt)), key = bucket * S^3 + tile-in-bucket.  The particles of a catalog are
// moved twice, each time by a counting sort whose workgroups stage their chunk
// in LDS ordered by key and then store it in per-key runs: first by bucket
// (few keys, long runs), then by tile inside the bucket.  Records are AoS:
// (px, py, pz) or (px, py, pz, w bits).
// count[key] += number of particles in the tile (LDS aggregation when it fits)
__global__ void __launch_bounds__(SORT_BLOCK) k_tile_count(const uint32_t* __restrict__ pos, int64_t n,
                                                           TileGeom g, int ntiles,
                                                           uint32_t* __restrict__ count) {
  extern __shared__ uint32_t lcount[];
  const bool lds = ntiles <= LDS_TILES_MAX;
  const int64_t chunk = (int64_t)SORT_BLOCK * SORT_PER_THREAD;
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = min(n, i0 + chunk);
  if (lds) {
    for (int t = threadIdx.x; t < ntiles; t += blockDim.x) lcount[t] = 0;
    __syncthreads();
  }
  for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    const int t = tile_key(pos[i], pos[n + i], pos[2 * n + i], g);
    if (lds) atomicAdd(&lcount[t], 1u);
    else atomicAdd(&count[t], 1u);
  }
  if (lds) {
    __syncthreads();
    for (int t = threadIdx.x; t < ntiles; t += blockDim.x) {
      const uint32_t c = lcount[t];
      if (c) atomicAdd(&count[t], c);
    }
  }
}

// Exclusive scan of R values by a workgroup of NT threads: emit(r, sum_{q < r}
// in[q]) for every r, each thread handling a run of consecutive r.  Wave
// prefix sums plus one LDS slot per wave (wsum, NT / 64 entries).
template <int NT, typename U, typename Emit>
__device__ void block_exclusive_scan(const U* in, int R, uint32_t* wsum, Emit emit) {
  const int per = (R + NT - 1) / NT;
  const int t0 = threadIdx.x * per, t1 = min(R, t0 + per);
  uint32_t s = 0;
  for (int t = t0; t < t1; ++t) s += in[t];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t v = s;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(v, off, 64);
    if (lane >= off) v += u;
  }
  if (lane == 63) wsum[wv] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int k = 0; k < NT / 64; ++k) {
      const uint32_t c = wsum[k];
      wsum[k] = run;
      run += c;
    }
  }
  __syncthreads();
  uint32_t run = wsum[wv] + v - s;
  for (int t = t0; t < t1; ++t) {
    emit(t, run);
    run += in[t];
  }
}

// Exclusive scan of the tile counts by one workgroup of 1024 threads: start =
// cursor = scan, and with bcur the bucket cursors bcur[b] = start[b << bshift].  Slabs of 4096 U tiles,
// 4 U consecutive ones per thread as 16-byte loads that are all in flight at
// once (one load at a time took 75 us for the 32768 tiles of a 512^3 mesh, two
// slabs of U = 4 take 13); ntiles is a power of 8 from 512 up (meshes of one bucket
// have k_small_scan), the arrays are 256-byte aligned.
template <int U>
__device__ __forceinline__ void tile_scan(const uint32_t* __restrict__ count, int ntiles, int bshift,
                                          uint32_t* __restrict__ start, uint32_t* __restrict__ cursor,
                                          uint32_t* __restrict__ bcur, uint32_t* wsum) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t base = 0;
  for (int t0 = 0; t0 < ntiles; t0 += 4096 * U) {
    const int t = t0 + (int)threadIdx.x * 4 * U;
    uint32_t c[4 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint4 q = make_uint4(0u, 0u, 0u, 0u);
      if (t + 4 * u < ntiles) q = *reinterpret_cast<const uint4*>(count + t + 4 * u);
      c[4 * u] = q.x; c[4 * u + 1] = q.y; c[4 * u + 2] = q.z; c[4 * u + 3] = q.w;
    }
    uint32_t s = 0;
#pragma unroll
    for (int e = 0; e < 4 * U; ++e) s += c[e];
    uint32_t v = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t u = __shfl_up(v, off, 64);
      if (lane >= off) v += u;
    }
    if (t0) __syncthreads();  // wsum of the previous slab is read
    if (lane == 63) wsum[wv] = v;
    __syncthreads();
    uint32_t w = wsum[lane & 15];  // inclusive scan of the 16 wave totals in every wavefront
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      const uint32_t u = __shfl_up(w, off, 16);
      if ((lane & 15) >= off) w += u;
    }
    uint32_t run = base + v - s + (wv ? __shfl(w, wv - 1, 64) : 0u);
    base += __shfl(w, 15, 64);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint4 q;
      q.x = run; run += c[4 * u];
      q.y = run; run += c[4 * u + 1];
      q.z = run; run += c[4 * u + 2];
      q.w = run; run += c[4 * u + 3];
      const int tt = t + 4 * u;
      if (tt < ntiles) {
        *reinterpret_cast<uint4*>(start + tt) = q;
        *reinterpret_cast<uint4*>(cursor + tt) = q;
      }
      if (bcur) {
        const uint32_t r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (tt + e < ntiles && ((tt + e) & ((1 << bshift) - 1)) == 0) bcur[(tt + e) >> bshift] = r[e];
      }
    }
  }
}

template <int U>
__global__ void __launch_bounds__(1024) k_tile_scan(const uint32_t* __restrict__ count, int ntiles,
                                                    int bshift, uint32_t* __restrict__ start,
                                                    uint32_t* __restrict__ cursor,
                                                    uint32_t* __restrict__ bcur) {
  __shared__ uint32_t wsum[16];
  tile_scan<U>(count, ntiles, bshift, start, cursor, bcur, wsum);
}

// k_tile_scan (workgroup 0) and, in workgroups 1 .. CNPC_SUMS_LEN, the
// fixed-order column sums of k_reduce_partials (first wavefront): the two
// steps between the first and the second sort step of a fused sort, one launch.
template <int U>
__global__ void __launch_bounds__(1024) k_tile_scan_sums(const uint32_t* __restrict__ count, int ntiles,
                                                         uint32_t* __restrict__ start,
                                                         uint32_t* __restrict__ cursor,
                                                         const double* __restrict__ partial, int nblocks,
                                                         double* __restrict__ sums) {
  __shared__ uint32_t wsum[16];
  if (blockIdx.x == 0) {
    tile_scan<U>(count, ntiles, 0, start, cursor, nullptr, wsum);
    return;
  }
  if (threadIdx.x >= 64) return;
  const int q = blockIdx.x - 1;
  double v = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += 64) v += partial[(int64_t)b * CNPC_SUMS_LEN + q];
  v = wave_sum(v);
  if (threadIdx.x == 0) sums[q] = v;
}

// zeroes p[0, n) and q[0, m) in one launch
__global__ void k_zero2_u32(uint32_t* p, int64_t n, uint32_t* q, int64_t m) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n + m; i += (int64_t)gridDim.x * blockDim.x) {
    if (i < n) p[i] = 0u;
    else q[i - n] = 0u;
  }
}

// Size in bytes of the LDS layout of k_partition with nt threads.
__host__ __device__ constexpr size_t partition_lds(int per, int rs, int rcap, int nt) {
  return (size_t)nt * per * (rs * 4 + 2) + (size_t)3 * rcap * 4 + 64;
}

// One counting-sort step over a chunk of NT * PER particles.
// FINE == false: input is the catalog (pos [3][n], optional w), key = bucket (rcap =
// number of buckets).
// FINE == true: input is records in bucket order, key = tile key; the chunk's keys lie
// in [bucket(first) S^3, (bucket(last) + 1) S^3); if that range is wider than
// rcap the chunk takes one global atomic per particle instead.
// cursor[key] hands out output slots (initialised to the key's start).
template <bool FINE, int RS, int PER, int NT>
__global__ void __launch_bounds__(NT) k_partition(const uint32_t* __restrict__ pos,
                                                            const float* __restrict__ w,
                                                            const Rec<RS>* __restrict__ rin,
                                                            int64_t n, TileGeom g, int rcap,
                                                            uint32_t* __restrict__ cursor,
                                                            Rec<RS>* __restrict__ rout, bool pack) {
  constexpr int CH = NT * PER;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Rec<RS>* stage = reinterpret_cast<Rec<RS>*>(smem_raw);                        // [CH]
  uint16_t* skey = reinterpret_cast<uint16_t*>(smem_raw + (size_t)CH * RS * 4);  // [CH]
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem_raw + (size_t)CH * (RS * 4 + 2));
  uint32_t* lstart = hist + rcap;
  uint32_t* gbase = lstart + rcap;
  uint32_t* wsum = gbase + rcap;  // 16 slots
  const int64_t c0 = (int64_t)blockIdx.x * CH;
  const int bshift = 3 * g.ls;
  int klo = 0, R;
  if (FINE) {
    const Rec<RS> a = rin[c0], b = rin[min(n, c0 + CH) - 1];
    const int kb0 = tile_key(a.v[0], a.v[1], a.v[2], g) >> bshift;
    const int kb1 = tile_key(b.v[0], b.v[1], b.v[2], g) >> bshift;
    klo = kb0 << bshift;
    R = (kb1 - kb0 + 1) << bshift;
  } else {
    R = rcap;
  }
  Rec<RS> r[PER];
  int key[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t i = c0 + (int64_t)k * NT + threadIdx.x;
    key[k] = -1;
    if (i < n) {
      if (FINE) {
        r[k] = rin[i];
      } else {
        r[k].v[0] = pos[i];
        r[k].v[1] = pos[n + i];
        r[k].v[2] = pos[2 * n + i];
        if constexpr (RS == 4) r[k].v[3] = __float_as_uint(w[i]);
      }
      const int t = tile_key(r[k].v[0], r[k].v[1], r[k].v[2], g);
      key[k] = FINE ? t - klo : (t >> bshift);
    }
  }
  if (FINE && R > rcap) {
    // wide key range: one global slot per particle
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (key[k] >= 0) put_rec(rout, atomicAdd(&cursor[klo + key[k]], 1u), r[k], FINE && pack, g.shift);
    return;
  }
  for (int t = threadIdx.x; t < R; t += NT) hist[t] = 0u;
  __syncthreads();
  uint32_t rank[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (key[k] >= 0) rank[k] = atomicAdd(&hist[key[k]], 1u);
  __syncthreads();
  block_exclusive_scan<NT>(hist, R, wsum, [&](int t, uint32_t v) {
    lstart[t] = v;
    const uint32_t c = hist[t];
    gbase[t] = c ? atomicAdd(&cursor[klo + t], c) : 0u;
  });
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (key[k] >= 0) {
      const uint32_t slot = lstart[key[k]] + rank[k];
      stage[slot] = r[k];
      skey[slot] = (uint16_t)key[k];
    }
  __syncthreads();
  const int cnt = (int)min((int64_t)CH, n - c0);
  for (int j = threadIdx.x; j < cnt; j += NT) {
    const int kk = skey[j];
    put_rec(rout, gbase[kk] + (j - lstart[kk]), stage[j], FINE && pack, g.shift);
  }
}

// The one sort step of a mesh of one tile bucket, both catalogs in one launch:
// workgroup b sorts the particles of sums workgroup b (every nblk-th run of 1024),
// whose place in every tile k_small_scan has left in hist[b], PER runs at a time (a cursor per tile in LDS; one
// atomic per chunk and tile on 64 shared counters took 25 us for 2.2e6 particles,
// 15 us here).
template <int RS, int PER>
__global__ void __launch_bounds__(1024) k_partition2(SmallPair sp, TileGeom g, int ntiles) {
  constexpr int NT = 1024, CH = NT * PER;
  const SmallCat c = sp.c[blockIdx.y];
  if ((int)blockIdx.x >= c.nblk) return;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Rec<RS>* stage = reinterpret_cast<Rec<RS>*>(smem_raw);                        // [CH]
  uint16_t* skey = reinterpret_cast<uint16_t*>(smem_raw + (size_t)CH * RS * 4);  // [CH]
  __shared__ uint32_t hist[SMALL_TILES], lstart[SMALL_TILES], gbase[SMALL_TILES];
  Rec<RS>* rout = reinterpret_cast<Rec<RS>*>(c.rec);
  static_assert(NT == SUMS_THREADS, "runs of the sums pass");
  const int64_t stride = (int64_t)c.nblk * NT;
  if (threadIdx.x < SMALL_TILES) {
    gbase[threadIdx.x] = (int)threadIdx.x < ntiles ? c.hist[(int64_t)blockIdx.x * SMALL_TILES + threadIdx.x] : 0u;
    hist[threadIdx.x] = 0u;
  }
  __syncthreads();
  for (int64_t c0 = (int64_t)blockIdx.x * NT; c0 < c.n; c0 += PER * stride) {
    Rec<RS> r[PER];
    int key[PER];
    uint32_t rank[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {  // clamped straight-line loads, all in flight at once
      const int64_t i = min(c0 + k * stride + threadIdx.x, c.n - 1);
      r[k].v[0] = c.pos[i];
      r[k].v[1] = c.pos[c.n + i];
      r[k].v[2] = c.pos[2 * c.n + i];
      if constexpr (RS == 4) r[k].v[3] = __float_as_uint(c.w[i]);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      key[k] = c0 + k * stride + threadIdx.x < c.n ? tile_key(r[k].v[0], r[k].v[1], r[k].v[2], g) : -1;
      if (key[k] >= 0) rank[k] = atomicAdd(&hist[key[k]], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 64) {  // exclusive scan of the chunk's histogram
      const uint32_t h = hist[threadIdx.x];
      uint32_t run = h;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(run, off, 64);
        if ((int)threadIdx.x >= off) run += u;
      }
      lstart[threadIdx.x] = run - h;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (key[k] >= 0) {
        const uint32_t slot = lstart[key[k]] + rank[k];
        stage[slot] = r[k];
        skey[slot] = (uint16_t)key[k];
      }
    __syncthreads();
    const int cnt = (int)(lstart[SMALL_TILES - 1] + hist[SMALL_TILES - 1]);
    for (int j = threadIdx.x; j < cnt; j += NT) {
      const int kk = skey[j];
      rout[gbase[kk] + (j - lstart[kk])] = stage[j];
    }
    __syncthreads();
    if (threadIdx.x < SMALL_TILES) {
      gbase[threadIdx.x] += hist[threadIdx.x];
      hist[threadIdx.x] = 0u;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------ fused bucket pass --
// One read of a catalog does the FP64 l = 0 catalog sums, the tile histogram and
// the first counting-sort step.  (Y_lm sums take a read of their own: formed
// here, between the barriers of the sort, their FP64 arithmetic cost more than
// that read, 476 against 199 + 140 us for 3.0e7 particles, 4.9 against
// 2.5 + 1.3 ms for 3.3e8.)  Buckets have a fixed capacity `cap` (bucket b at
// region + b cap): a workgroup reserves its run in bucket b with one atomic on
// bcnt[b] and sends whatever would pass the capacity to the overflow region
// (reserved on *ovf), which the tile pass takes as chunks of mixed buckets.
// Persistent workgroups walk chunks of NT * PER particles, so the LDS tile
// histogram is flushed with one atomic per non-empty tile per workgroup; with
// more tiles than LDS_TILES_MAX k_region_count counts them afterwards.  With
// `pack` (FP32 painter, unweighted, 256^3 and more, at most 2^16 tiles) a
// record goes out as pack_rec in 8 bytes and its tile index in 2 more, in an
// array after the 8-byte records of its region (both fit the 12-byte records'
// room); the LDS then also stages each record's tile index after the tile
// histogram.
struct BucketArgs {
  TileGeom g;
  int ntiles, nbuckets;
  uint32_t cap;       // records per bucket region
  uint32_t* bcnt;     // [nbuckets] reservations per bucket (may exceed cap)
  uint32_t* ovf;      // overflow records reserved
  uint32_t* tcount;   // [ntiles] tile histogram (filled here up to LDS_TILES_MAX tiles)
  double* partial;    // [gridDim.x][CNPC_SUMS_LEN] catalog-sum partials
  bool pack;          // records out as pack_rec + a 16-bit tile index (rkey / okey)
  uint16_t* rkey;     // [nbuckets * cap] tile index of each region record (pack)
  uint16_t* okey;     // [n] tile index of each overflow record (pack)
};

// LDS bytes of k_bucket_pass
__host__ __device__ constexpr size_t bucket_pass_lds(int per, int rs, int nbuckets, int nt, int ltiles) {
  return (size_t)nt * per * (rs * 4 + 2) + (size_t)6 * nbuckets * 4 + 64 + (size_t)ltiles * 4;
}

// PF: the next chunk's particles are loaded while the current one is sorted
template <int RS, int PER, int NT, bool PF>
__global__ void __launch_bounds__(NT) k_bucket_pass(const uint32_t* __restrict__ pos, const float* __restrict__ w,
                                                    int64_t n, SumsArgs sa, BucketArgs ba,
                                                    Rec<RS>* __restrict__ region, Rec<RS>* __restrict__ ovf_out) {
  constexpr int CH = NT * PER;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Rec<RS>* stage = reinterpret_cast<Rec<RS>*>(smem_raw);                        // [CH]
  uint16_t* skey = reinterpret_cast<uint16_t*>(smem_raw + (size_t)CH * RS * 4);  // [CH]
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem_raw + (size_t)CH * (RS * 4 + 2));
  uint32_t* lstart = hist + ba.nbuckets;
  uint32_t* gbase = lstart + ba.nbuckets;
  uint32_t* nin = gbase + ba.nbuckets;
  uint32_t* obase = nin + ba.nbuckets;
  uint32_t* wsum = obase + ba.nbuckets;  // 16 slots
  uint32_t* ltile = wsum + 16;
  const bool lds_tiles = ba.ntiles <= LDS_TILES_MAX;
  if (lds_tiles)
    for (int t = threadIdx.x; t < ba.ntiles; t += NT) ltile[t] = 0u;
  double acc[CNPC_SUMS_LEN];
#pragma unroll
  for (int q = 0; q < CNPC_SUMS_LEN; ++q) acc[q] = 0.0;
  const double scale = sa.boxsize / 4294967296.0;
  const int bshift = 3 * ba.g.ls;
  const int64_t stride = (int64_t)gridDim.x * CH;
  // c < n: indices past the end are clamped to the last particle, so the
  // loads form straight-line code and are all in flight before the first use
  // (a load under a branch is waited for before the next one is issued)
  auto load_chunk = [&](int64_t c, Rec<RS>* dst) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int64_t i = min(c + (int64_t)k * NT + threadIdx.x, n - 1);
      dst[k].v[0] = pos[i];
      dst[k].v[1] = pos[n + i];
      dst[k].v[2] = pos[2 * n + i];
      if constexpr (RS == 4) dst[k].v[3] = __float_as_uint(w[i]);
    }
  };
  uint16_t* stile = reinterpret_cast<uint16_t*>(ltile + (lds_tiles ? ba.ntiles : 0));  // [CH] (pack)
  Rec<RS> rn[PF ? PER : 1];
  if constexpr (PF) load_chunk((int64_t)blockIdx.x * CH, rn);
  for (int64_t c0 = (int64_t)blockIdx.x * CH; c0 < n; c0 += stride) {
    Rec<RS> r[PER];
    int key[PER];
    __syncthreads();  // the previous chunk's LDS reads are done
    for (int t = threadIdx.x; t < ba.nbuckets; t += NT) hist[t] = 0u;
#pragma unroll
    for (int k = 0; k < PER; ++k) key[k] = -1;
    if constexpr (PF) {
#pragma unroll
      for (int k = 0; k < PER; ++k) r[k] = rn[k];
      if (c0 + stride < n) load_chunk(c0 + stride, rn);
    } else {
      load_chunk(c0, r);
    }
    __syncthreads();
    uint32_t rank[PER];
    int tk[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int64_t i = c0 + (int64_t)k * NT + threadIdx.x;
      tk[k] = 0;
      if (i < n) {
        const int t = tile_key(r[k].v[0], r[k].v[1], r[k].v[2], ba.g);
        tk[k] = t;
        key[k] = t >> bshift;
        if (lds_tiles) atomicAdd(&ltile[t], 1u);
        rank[k] = atomicAdd(&hist[key[k]], 1u);
        const double wi = RS == 4 ? (double)__uint_as_float(r[k].v[3]) : 1.0;
        sums_add<0>(acc, r[k].v[0], r[k].v[1], r[k].v[2], wi, scale, sa);
      }
    }
    __syncthreads();
    block_exclusive_scan<NT>(hist, ba.nbuckets, wsum, [&](int b, uint32_t v) {
      lstart[b] = v;
      const uint32_t c = hist[b];
      uint32_t gb = 0u, ni = 0u, ob = 0u;
      if (c) {
        gb = atomicAdd(&ba.bcnt[b], c);
        ni = gb >= ba.cap ? 0u : min(c, ba.cap - gb);
        if (c > ni) ob = atomicAdd(ba.ovf, c - ni);
      }
      gbase[b] = gb;
      nin[b] = ni;
      obase[b] = ob;
    });
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (key[k] >= 0) {
        const uint32_t slot = lstart[key[k]] + rank[k];
        stage[slot] = r[k];
        skey[slot] = (uint16_t)key[k];
        if (ba.pack) stile[slot] = (uint16_t)tk[k];
      }
    __syncthreads();
    const int cnt = (int)min((int64_t)CH, n - c0);
    if (RS == 3 && ba.pack) {
      for (int j = threadIdx.x; j < cnt; j += NT) {
        const int b = skey[j];
        const uint32_t q = (uint32_t)j - lstart[b];
        const uint64_t v = pack_rec(*reinterpret_cast<const Rec<3>*>(&stage[j]), ba.g.shift);
        if (q < nin[b]) {
          const int64_t o = (int64_t)b * ba.cap + gbase[b] + q;
          reinterpret_cast<uint64_t*>(region)[o] = v;
          ba.rkey[o] = stile[j];
        } else {
          const int64_t o = obase[b] + (q - nin[b]);
          reinterpret_cast<uint64_t*>(ovf_out)[o] = v;
          ba.okey[o] = stile[j];
        }
      }
    } else {
      for (int j = threadIdx.x; j < cnt; j += NT) {
        const int b = skey[j];
        const uint32_t q = (uint32_t)j - lstart[b];
        if (q < nin[b]) region[(int64_t)b * ba.cap + gbase[b] + q] = stage[j];
        else ovf_out[obase[b] + (q - nin[b])] = stage[j];
      }
    }
  }
  // catalog-sum partial of the workgroup (fixed-order reduction)
  __syncthreads();
  double* red = reinterpret_cast<double*>(smem_raw);  // [NT / 64][CNPC_SUMS_LEN], over the stage
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < CNPC_SUMS_LEN; ++q) {
    const double v = q < sums_used(0) ? wave_sum(acc[q]) : 0.0;
    if (lane == 0) red[wv * CNPC_SUMS_LEN + q] = v;
  }
  __syncthreads();
  if (threadIdx.x < CNPC_SUMS_LEN) {
    double v = 0.0;
    for (int k = 0; k < NT / 64; ++k) v += red[k * CNPC_SUMS_LEN + threadIdx.x];
    ba.partial[(int64_t)blockIdx.x * CNPC_SUMS_LEN + threadIdx.x] = v;
  }
  if (lds_tiles)
    for (int t = threadIdx.x; t < ba.ntiles; t += NT) {
      const uint32_t c = ltile[t];
      if (c) atomicAdd(&ba.tcount[t], c);
    }
}

// Overflow records lie in runs of one bucket, one per (workgroup, chunk, bucket)
// of the bucket pass, so a chunk of them holds few buckets.  The passes over them
// number the buckets of a chunk (the first OVF_SLOTS in key order; the rest take
// global atomics) and count and sort in LDS by (bucket number, tile in bucket),
// as the region chunks do.  A catalog that fills a part of its box has most of its
// records here: with one global atomic per record 2.2e7 particles in 1 / 64 of a
// 256^3 box took 34 ms (FP64 P_0 pass) before, 2.8 here, in 1 / 8 of it 6.1 ms
// before, 1.8 here.
constexpr int OVF_SLOTS = 32;

// flag, slot: [nbuckets]; list: [nslots].  Numbers the buckets tk[k] >> bshift
// (tk[k] >= 0) of a chunk: slot[b] (255 past the first nslots), list[slot] = b.
// Starts and ends with a workgroup barrier.
template <int NT, int PER>
__device__ __forceinline__ void number_buckets(const int* tk, int bshift, int nbuckets, int nslots, uint8_t* flag,
                                               uint8_t* slot, uint32_t* list, uint32_t* wsum) {
  __syncthreads();
  for (int b = threadIdx.x; b < nbuckets; b += NT) flag[b] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (tk[k] >= 0) flag[tk[k] >> bshift] = 1;
  __syncthreads();
  block_exclusive_scan<NT>(flag, nbuckets, wsum, [&](int b, uint32_t v) {
    if (!flag[b]) return;
    slot[b] = (uint8_t)(v < (uint32_t)nslots ? v : 255u);
    if (v < (uint32_t)nslots) list[v] = b;
  });
  __syncthreads();
}

// records per thread of an overflow chunk of a tile pass with per ones (the tables
// leave two workgroups per CU whole chunks of 8-byte records, half chunks of others)
__host__ __device__ constexpr int ovf_per(int per, int vbytes) { return per > 1 && vbytes > 8 ? per / 2 : per; }
// LDS bytes of sort_overflow
__host__ __device__ constexpr size_t overflow_lds(int per, int vbytes, int nt, int nbuckets, int bshift) {
  return (size_t)nt * per * (vbytes + 2) + (size_t)4 * (3 * (OVF_SLOTS << bshift) + OVF_SLOTS + 16) + 2 * (size_t)nbuckets;
}

// Tile step over the overflow records c0 .. (one workgroup's share): load(c, i, v)
// reads record c + i and returns its tile, put(o, v) writes one to output slot o.
template <int NT, int PER, typename V, typename Load, typename Put>
__device__ __forceinline__ void sort_overflow(int64_t c0, int64_t stride, uint32_t no, int nbuckets, int bshift,
                                              uint32_t* __restrict__ cursor, unsigned char* smem, Load load, Put put) {
  constexpr int CH = NT * PER;
  const int R = OVF_SLOTS << bshift, mask = (1 << bshift) - 1;
  V* stage = reinterpret_cast<V*>(smem);                                          // [CH]
  uint16_t* skey = reinterpret_cast<uint16_t*>(smem + (size_t)CH * sizeof(V));     // [CH]
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem + (size_t)CH * (sizeof(V) + 2));  // [R] each
  uint32_t *lstart = hist + R, *gbase = lstart + R;
  uint32_t* list = gbase + R;       // [OVF_SLOTS]
  uint32_t* wsum = list + OVF_SLOTS;  // 16 slots
  uint8_t *flag = reinterpret_cast<uint8_t*>(wsum + 16), *slot = flag + nbuckets;
  if (c0 >= no) return;
  V rn[PER];  // the next chunk, loaded while the current one is sorted (clamped indices)
  int tn[PER];
  auto load_chunk = [&](int64_t c) {
    const int last = (int)min((int64_t)CH, no - c) - 1;
#pragma unroll
    for (int k = 0; k < PER; ++k) tn[k] = load(c, (uint32_t)min(k * NT + (int)threadIdx.x, last), rn[k]);
  };
  load_chunk(c0);
  for (; c0 < no; c0 += stride) {
    V r[PER];
    int tk[PER];  // tile, then (bucket number, tile in bucket) | rank << 16; < 0: none
    const int cin = (int)min((int64_t)CH, no - c0);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      r[k] = rn[k];
      tk[k] = k * NT + (int)threadIdx.x < cin ? tn[k] : -1;
    }
    if (c0 + stride < no) load_chunk(c0 + stride);
    number_buckets<NT, PER>(tk, bshift, nbuckets, OVF_SLOTS, flag, slot, list, wsum);
    for (int t = threadIdx.x; t < R; t += NT) hist[t] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (tk[k] < 0) continue;
      const int b = slot[tk[k] >> bshift];
      if (b < OVF_SLOTS) {
        tk[k] = (b << bshift) | (tk[k] & mask);
        tk[k] |= (int)(atomicAdd(&hist[tk[k]], 1u) << 16);
      } else {
        put(atomicAdd(&cursor[tk[k]], 1u), r[k]);
        tk[k] = -1;
      }
    }
    __syncthreads();
    block_exclusive_scan<NT>(hist, R, wsum, [&](int t, uint32_t v) {
      lstart[t] = v;
      const uint32_t c = hist[t];
      gbase[t] = c ? atomicAdd(&cursor[(list[t >> bshift] << bshift) | (t & mask)], c) : 0u;
    });
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (tk[k] >= 0) {
        const uint32_t j = lstart[tk[k] & 0xffff] + (uint32_t)(tk[k] >> 16);
        stage[j] = r[k];
        skey[j] = (uint16_t)tk[k];
      }
    __syncthreads();
    const int cnt = (int)(lstart[R - 1] + hist[R - 1]);
    for (int j = threadIdx.x; j < cnt; j += NT) {
      const int kk = skey[j];
      put(gbase[kk] + (j - lstart[kk]), stage[j]);
    }
  }
}

// Tile histogram of bucket-sorted records, for meshes of more tiles than the
// bucket pass holds in LDS (512^3 and more).  A bucket's records fall into its
// own S^3 <= 64 tiles, so a workgroup counts REGION_CHUNK of them in LDS (one
// copy per wavefront) and adds each tile once; the overflow records are counted
// by the buckets of a chunk.  Bound by its reads: the 16-bit tile indices of packed
// records (2 bytes a particle) or the records themselves (12 or 16).  One
// global atomic per particle in the bucket pass, which it replaces, held that
// pass to 2.6 ms for 5.5e7 particles (0.90 ms without it, and 0.04 ms here; 3.3e8
// full records: 0.80 ms here).
constexpr int REGION_CHUNK = 65536;
constexpr int COUNT_PER = 8, COUNT_SLOTS = 64;  // overflow chunks: records per thread, buckets
__host__ __device__ constexpr size_t region_count_lds(int nbuckets, int bshift) {
  return (size_t)4 * ((COUNT_SLOTS << bshift) + COUNT_SLOTS + 16) + 2 * (size_t)nbuckets;
}
template <int RS>
__global__ void __launch_bounds__(1024) k_region_count(const Rec<RS>* __restrict__ region,
                                                       const uint16_t* __restrict__ rkey,
                                                       const Rec<RS>* __restrict__ ovf_in,
                                                       const uint16_t* __restrict__ okey,
                                                       const uint32_t* __restrict__ bcnt,
                                                       const uint32_t* __restrict__ ovf, uint32_t cap,
                                                       int chunks_per_bucket, int nbuckets, TileGeom g, bool packed,
                                                       uint32_t* __restrict__ count) {
  __shared__ uint32_t hist[16][64];
  const int nreg = nbuckets * chunks_per_bucket;
  if ((int)blockIdx.x >= nreg) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int bshift = 3 * g.ls, R = COUNT_SLOTS << bshift, mask = (1 << bshift) - 1;
    uint32_t* oh = reinterpret_cast<uint32_t*>(smem_raw);  // [R]
    uint32_t *list = oh + R, *wsum = list + COUNT_SLOTS;
    uint8_t *flag = reinterpret_cast<uint8_t*>(wsum + 16), *slot = flag + nbuckets;
    const uint32_t no = *ovf;
    constexpr int64_t CH = 1024 * COUNT_PER;
    for (int64_t c0 = (int64_t)(blockIdx.x - nreg) * CH; c0 < no; c0 += (int64_t)(gridDim.x - nreg) * CH) {
      int tk[COUNT_PER];
#pragma unroll
      for (int k = 0; k < COUNT_PER; ++k) {
        const int64_t i = c0 + k * 1024 + (int)threadIdx.x, ii = min(i, (int64_t)no - 1);
        if (packed) tk[k] = okey[ii];
        else tk[k] = tile_key(ovf_in[ii].v[0], ovf_in[ii].v[1], ovf_in[ii].v[2], g);
        if (i >= no) tk[k] = -1;
      }
      number_buckets<1024, COUNT_PER>(tk, bshift, nbuckets, COUNT_SLOTS, flag, slot, list, wsum);
      for (int t = threadIdx.x; t < R; t += 1024) oh[t] = 0u;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < COUNT_PER; ++k) {
        if (tk[k] < 0) continue;
        const int b = slot[tk[k] >> bshift];
        if (b < COUNT_SLOTS) atomicAdd(&oh[(b << bshift) | (tk[k] & mask)], 1u);
        else atomicAdd(&count[tk[k]], 1u);
      }
      __syncthreads();
      for (int t = threadIdx.x; t < R; t += 1024) {
        const uint32_t c = oh[t];
        if (c) atomicAdd(&count[(list[t >> bshift] << bshift) | (t & mask)], c);
      }
    }
    return;
  }
  const int b = blockIdx.x / chunks_per_bucket, jc = blockIdx.x - b * chunks_per_bucket;
  const uint32_t nb_ = min(bcnt[b], cap), c0 = (uint32_t)jc * REGION_CHUNK;
  if (c0 >= nb_) return;
  const uint32_t c1 = min(nb_, c0 + REGION_CHUNK);
  const int wv = threadIdx.x >> 6, klo = b << (3 * g.ls);
  hist[wv][threadIdx.x & 63] = 0u;
  const int64_t o = (int64_t)b * cap;
  constexpr int U = 4;  // independent loads per trip, indices clamped to the last record
  for (uint32_t i0 = c0 + threadIdx.x; i0 < c1; i0 += 1024u * U) {
    int t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = min(i0 + 1024u * u, c1 - 1u);
      if (packed) {
        t[u] = rkey[o + i];
      } else {
        const Rec<RS> r = region[o + i];
        t[u] = tile_key(r.v[0], r.v[1], r.v[2], g);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + 1024u * u < c1) atomicAdd(&hist[wv][t[u] - klo], 1u);
  }
  __syncthreads();
  if (threadIdx.x < 64u && (int)threadIdx.x < 1 << (3 * g.ls)) {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) c += hist[k][threadIdx.x];
    if (c) atomicAdd(&count[klo + threadIdx.x], c);
  }
}

// The tile step over the overflow records (a launch of its own: inside the tile pass
// its registers and tables cost the region chunks of a batch's streams 3% of the whole
// batch).  PACKED: 8-byte records (pack_rec) with their tile index in okey, else Rec<RS>,
// in chunks of half the size: the tables take the other half of the LDS.
template <int RS, int PER, int NT, bool PACKED>
__global__ void __launch_bounds__(NT, 8) k_overflow_pass(const void* __restrict__ ovf_in,
                                                         const uint16_t* __restrict__ okey,
                                                         const uint32_t* __restrict__ ovf, int nbuckets, TileGeom g,
                                                         uint32_t* __restrict__ cursor, void* __restrict__ rout,
                                                         bool pack) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int bshift = 3 * g.ls;
  const int64_t c0 = (int64_t)blockIdx.x * NT * PER, stride = (int64_t)gridDim.x * NT * PER;
  if constexpr (PACKED) {
    const uint64_t* in = reinterpret_cast<const uint64_t*>(ovf_in);
    uint64_t* out = reinterpret_cast<uint64_t*>(rout);
    sort_overflow<NT, PER, uint64_t>(
        c0, stride, *ovf, nbuckets, bshift, cursor, smem_raw,
        [&](int64_t c, uint32_t i, uint64_t& v) {
          v = (in + c)[i];
          return (int)(okey + c)[i];
        },
        [&](uint32_t o, uint64_t v) { out[o] = v; });
  } else {
    const Rec<RS>* in = reinterpret_cast<const Rec<RS>*>(ovf_in);
    Rec<RS>* out = reinterpret_cast<Rec<RS>*>(rout);
    sort_overflow<NT, PER, Rec<RS>>(
        c0, stride, *ovf, nbuckets, bshift, cursor, smem_raw,
        [&](int64_t c, uint32_t i, Rec<RS>& v) {
          v = (in + c)[i];
          return tile_key(v.v[0], v.v[1], v.v[2], g);
        },
        [&](uint32_t o, const Rec<RS>& v) { put_rec(out, o, v, pack, g.shift); });
  }
}

// Second counting-sort step over the bucket regions: workgroup (b, j) sorts
// records j CH .. of bucket b (its keys lie in bucket b).
template <int RS, int PER, int NT>
__global__ void __launch_bounds__(NT) k_tile_pass(const Rec<RS>* __restrict__ region, const uint32_t* __restrict__ bcnt,
                                                  uint32_t cap, int chunks_per_bucket, TileGeom g,
                                                  uint32_t* __restrict__ cursor, Rec<RS>* __restrict__ rout, bool pack) {
  constexpr int CH = NT * PER;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int bshift = 3 * g.ls;
  const int R = 1 << bshift;  // tiles per bucket
  const int b = blockIdx.x / chunks_per_bucket, jc = blockIdx.x - b * chunks_per_bucket;
  const uint32_t nb_ = min(bcnt[b], cap);
  const int64_t c0 = (int64_t)jc * CH;
  if (c0 >= nb_) return;
  const int cnt = (int)min((int64_t)CH, (int64_t)nb_ - c0);
  const Rec<RS>* rin = region + (int64_t)b * cap + c0;
  Rec<RS>* stage = reinterpret_cast<Rec<RS>*>(smem_raw);                        // [CH]
  uint16_t* skey = reinterpret_cast<uint16_t*>(smem_raw + (size_t)CH * RS * 4);  // [CH]
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem_raw + (size_t)CH * (RS * 4 + 2));
  uint32_t* lstart = hist + R;
  uint32_t* gbase = lstart + R;
  uint32_t* wsum = gbase + R;  // 16 slots
  const int klo = b << bshift;
  Rec<RS> r[PER];
  int key[PER];
  // cnt >= 1: clamped straight-line loads, all in flight before the first use
#pragma unroll
  for (int k = 0; k < PER; ++k) r[k] = rin[min(k * NT + (int)threadIdx.x, cnt - 1)];
#pragma unroll
  for (int k = 0; k < PER; ++k)
    key[k] = k * NT + (int)threadIdx.x < cnt ? tile_key(r[k].v[0], r[k].v[1], r[k].v[2], g) - klo : -1;
  for (int t = threadIdx.x; t < R; t += NT) hist[t] = 0u;
  __syncthreads();
  uint32_t rank[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (key[k] >= 0) rank[k] = atomicAdd(&hist[key[k]], 1u);
  __syncthreads();
  block_exclusive_scan<NT>(hist, R, wsum, [&](int t, uint32_t v) {
    lstart[t] = v;
    const uint32_t c = hist[t];
    gbase[t] = c ? atomicAdd(&cursor[klo + t], c) : 0u;
  });
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (key[k] >= 0) {
      const uint32_t slot = lstart[key[k]] + rank[k];
      stage[slot] = r[k];
      skey[slot] = (uint16_t)key[k];
    }
  __syncthreads();
  for (int j = threadIdx.x; j < cnt; j += NT) {
    const int kk = skey[j];
    put_rec(rout, gbase[kk] + (j - lstart[kk]), stage[j], pack, g.shift);
  }
}

// k_tile_pass over records the bucket pass wrote packed (pack_rec + 16-bit tile
// index, for the FP32 painter): the tile index comes from its own array and the
// packed records are moved as they are
template <int PER, int NT>
__global__ void __launch_bounds__(NT) k_tile_pass_packed(const uint64_t* __restrict__ region,
                                                         const uint16_t* __restrict__ rkey,
                                                         const uint32_t* __restrict__ bcnt, uint32_t cap,
                                                         int chunks_per_bucket, TileGeom g,
                                                         uint32_t* __restrict__ cursor, uint64_t* __restrict__ rout) {
  constexpr int CH = NT * PER;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int bshift = 3 * g.ls;
  const int R = 1 << bshift;
  const int b = blockIdx.x / chunks_per_bucket, jc = blockIdx.x - b * chunks_per_bucket;
  const uint32_t nb_ = min(bcnt[b], cap);
  const int64_t c0 = (int64_t)jc * CH;
  if (c0 >= nb_) return;
  const int cnt = (int)min((int64_t)CH, (int64_t)nb_ - c0);
  const uint64_t* rin = region + (int64_t)b * cap + c0;
  const uint16_t* kin = rkey + (int64_t)b * cap + c0;
  uint64_t* stage = reinterpret_cast<uint64_t*>(smem_raw);                  // [CH]
  uint16_t* skey = reinterpret_cast<uint16_t*>(smem_raw + (size_t)CH * 8);  // [CH]
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem_raw + (size_t)CH * 10);
  uint32_t* lstart = hist + R;
  uint32_t* gbase = lstart + R;
  uint32_t* wsum = gbase + R;  // 16 slots
  const int klo = b << bshift;
  uint64_t r[PER];
  int key[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int ii = min(k * NT + (int)threadIdx.x, cnt - 1);
    r[k] = rin[ii];
    key[k] = (int)kin[ii];
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) key[k] = k * NT + (int)threadIdx.x < cnt ? key[k] - klo : -1;
  for (int t = threadIdx.x; t < R; t += NT) hist[t] = 0u;
  __syncthreads();
  uint32_t rank[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (key[k] >= 0) rank[k] = atomicAdd(&hist[key[k]], 1u);
  __syncthreads();
  block_exclusive_scan<NT>(hist, R, wsum, [&](int t, uint32_t v) {
    lstart[t] = v;
    const uint32_t c = hist[t];
    gbase[t] = c ? atomicAdd(&cursor[klo + t], c) : 0u;
  });
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (key[k] >= 0) {
      const uint32_t slot = lstart[key[k]] + rank[k];
      stage[slot] = r[k];
      skey[slot] = (uint16_t)key[k];
    }
  __syncthreads();
  for (int j = threadIdx.x; j < cnt; j += NT) {
    const int kk = skey[j];
    rout[gbase[kk] + (j - lstart[kk])] = stage[j];
  }
}

// ------------------------------------------------------------------ paint --
// 1-D stencil: weights and the offset of the first node relative to the base
// cell c = floor(u), from the fraction bits (shift <= 28).  TSC phase A:
// i = floor(u + 1/2); phase B: i = floor(u) (u - 1/2 + 1/2).  CIC phase A: nodes
// c, c + 1; phase B: u - 1/2.
template <typename T, int ASSIGN>
__device__ __forceinline__ int stencil_1d(uint32_t p, int shift, int phase, T inv, T* wt) {
  const int one = 1 << shift, half = one >> 1;
  const int f = (int)(p & (uint32_t)(one - 1));
  const bool up = f >= half;
  if constexpr (ASSIGN == CNPC_TSC) {
    const T d = T(phase == 0 ? (up ? f - one : f) : f - half) * inv;
    const T a = T(0.5) - d, b = T(0.5) + d;
    wt[0] = T(0.5) * a * a;
    wt[1] = T(0.75) - d * d;
    wt[2] = T(0.5) * b * b;
    return phase == 0 ? (up ? 0 : -1) : -1;
  } else {
    const T d = T(phase == 0 ? f : (up ? f - half : f + half)) * inv;
    wt[0] = T(1) - d;
    wt[1] = d;
    return phase == 0 ? 0 : (up ? 0 : -1);
  }
}

// Tile-sorted catalogs of a painting launch (blockIdx.y; one, or the two of a
// mesh of one tile bucket); blocks[c], blocks[c + 2]: the w and w^2 blocks.
template <typename T, int RS>
struct PaintCats {
  const Rec<RS>* rec[2];
  const uint32_t *start[2], *count[2];
  T* blocks[4];
};

// Contributions are accumulated as 64-bit fixed point (2^-40 units) with
// integer LDS atomics: on gfx950 integer LDS atomics run at full rate while
// FP32 LDS atomics are an order of magnitude slower, and integer sums do not
// depend on the order in which the threads add (bit-reproducible blocks).
constexpr double FIX_SCALE = 1099511627776.0;  // 2^40
constexpr double FIX_INV = 1.0 / 1099511627776.0;
// |x| < 2^51: round(x) as a 64-bit integer, from the mantissa of x + 1.5 2^52 (one
// addition, rounding to nearest even, and one 32-bit subtraction; the
// conversion to a 64-bit integer takes a dozen instructions)
constexpr double FIX_MAGIC = 6755399441055744.0;
__device__ __forceinline__ unsigned long long fix_bits(double x_plus_magic) {
  const uint64_t b = (uint64_t)__double_as_longlong(x_plus_magic);
  return ((uint64_t)((uint32_t)(b >> 32) - 0x43380000u) << 32) | (uint32_t)b;
}

// adds one particle to the block; FAST: |weight| < 1024, so that every
// contribution is below 2^51 units
template <typename T, int ASSIGN, bool FAST>
__device__ __forceinline__ void paint_one(unsigned long long* __restrict__ acc, T wv, const T* wx, const T* wy,
                                          const T* wz, int a1, int a0) {
  constexpr int NP = ASSIGN == CNPC_TSC ? 3 : 2;
#pragma unroll
  for (int ix = 0; ix < NP; ++ix) {
    // FP64: the unit scale goes into the x weight (a power of two, exact)
    const T vx = sizeof(T) == 8 && FAST ? wv * wx[ix] * T(FIX_SCALE) : wv * wx[ix];
#pragma unroll
    for (int iy = 0; iy < NP; ++iy) {
      const T vxy = vx * wy[iy];
#pragma unroll
      for (int iz = 0; iz < NP; ++iz) {
        unsigned long long fix;
        if constexpr (!FAST) fix = (unsigned long long)__double2ll_rn((double)(vxy * wz[iz]) * FIX_SCALE);
        else if constexpr (sizeof(T) == 8) fix = fix_bits(__builtin_fma((double)vxy, (double)wz[iz], FIX_MAGIC));
        else fix = fix_bits(__builtin_fma((double)(vxy * wz[iz]), FIX_SCALE, FIX_MAGIC));
        atomicAdd(&acc[(iz == 0 ? a0 : a1) + ix * BW * BW + iy * BW + iz], fix);
      }
    }
  }
}

// A workgroup paints one tile, interlacing phase and weight power (w into
// blocks1, w^2 into blocks2; npow 1: w alone): its 55 KB block leaves room for
// two workgroups per CU, 8 wavefronts per SIMD (both phases in one workgroup
// left 4).  The workgroups of a tile are 8 apart in launch order, so that they
// run on one XCD and read its records from that L2.  Bound by the 64-bit LDS
// atomics (27 TSC or 8 CIC per particle, phase and power).  256^3 TSC
// interlaced, 3.0e7 particles: FP64 843 us with conversion calls and one
// workgroup per CU before, 669 us here; weighted FP32, 1.9e7 particles, both
// powers: 1270 us before, 961 us here.
template <typename T, int ASSIGN, int RS>
__global__ void __launch_bounds__(1024, 8) k_paint_tiles(PaintCats<T, RS> pc, TileGeom g, int nphase, int npow) {
  const Rec<RS>* __restrict__ rec = pc.rec[blockIdx.y];
  const uint32_t* __restrict__ start = pc.start[blockIdx.y];
  const uint32_t* __restrict__ count = pc.count[blockIdx.y];
  __shared__ __align__(16) unsigned long long acc[BVOL];
  const int nsub = nphase * npow;
  int t, sub;  // tile (tx * nt + ty) * nt + tz
  if (g.nt > 1) {
    t = (int)(blockIdx.x / (8u * nsub)) * 8 + (int)(blockIdx.x & 7u);
    sub = (int)(blockIdx.x >> 3) % nsub;
  } else {
    t = 0;
    sub = (int)blockIdx.x;
  }
  const int ph = nphase == 2 ? sub & 1 : 0, pw = nphase == 2 ? sub >> 1 : sub;
  const int shift = g.shift;
  for (int i = threadIdx.x; i < BVOL; i += 1024) acc[i] = 0ull;
  __syncthreads();
  const int key = key_of(t / (g.nt * g.nt), (t / g.nt) % g.nt, t % g.nt, g);
  const uint32_t s0 = start[key], cnt = count[key];
  const T inv = T(1) / T(1 << shift);
  for (uint32_t k = threadIdx.x; k < cnt; k += 1024u) {
    const Rec<RS> p = rec[(int64_t)s0 + k];
    T wv = T(1);
    if constexpr (RS == 4) {
      wv = T(__uint_as_float(p.v[3]));
      if (pw == 1) wv *= wv;
    }
    T wx[3], wy[3], wz[3];
    const int lx = ((int)(p.v[0] >> shift) & 15) + 1 + stencil_1d<T, ASSIGN>(p.v[0], shift, ph, inv, wx);
    const int ly = ((int)(p.v[1] >> shift) & 15) + 1 + stencil_1d<T, ASSIGN>(p.v[1], shift, ph, inv, wy);
    const int lz = ((int)(p.v[2] >> shift) & 15) + 1 + stencil_1d<T, ASSIGN>(p.v[2], shift, ph, inv, wz);
    // node lz + iz sits at lz + iz - 1 in its row, node 0 at 18
    const int a1 = lx * BW * BW + ly * BW + lz - 1;
    const int a0 = a1 + (lz == 0 ? BW : 0);
    if (RS == 3 || fabs(wv) < T(1024)) paint_one<T, ASSIGN, true>(acc, wv, wx, wy, wz, a1, a0);
    else paint_one<T, ASSIGN, false>(acc, wv, wx, wy, wz, a1, a0);
  }
  __syncthreads();
  T* out = pc.blocks[blockIdx.y + 2 * pw] + ((int64_t)t * nphase + ph) * BSTRIDE;
  for (int i = threadIdx.x; i < BVOL; i += 1024) out[i] = T((double)(long long)acc[i] * FIX_INV);
}

// Unit-weight FP32 painting with 32-bit LDS atomics.  Each round of the
// workgroup paints one particle per thread; a node then gains at most
// PPF * max node weight per flush interval (PPF = particles per flush), which
// at 2^21 units stays below 2^32 (TSC: 4096 * 0.421875 * 2^21; CIC:
// 1024 * 1 * 2^21), so the 32-bit sums are exact.  After every interval each
// thread moves the nodes it owns into 64-bit registers and clears them.  The
// result equals the 64-bit fixed-point sum of the contributions rounded to
// 2^-21 (half up), independent of the order of the additions.  From 256^3 up
// the particles come as packed 8-byte records (pack_rec): positions inside the
// tile on a 2^-17 cell grid.
constexpr int PAINT32_THREADS = 1024;
constexpr int PAINT32_OWN = (2 * BVOL + PAINT32_THREADS - 1) / PAINT32_THREADS;  // nodes per thread

// 1-D stencil in 32-bit integer arithmetic (shift <= 28): same nodes and
// weights as stencil_1d<float>, times `scale`, a power of two (scaling by it
// is exact, so a scaled weight is bit for bit the scaled unscaled weight).
template <int ASSIGN>
__device__ __forceinline__ int stencil32(uint32_t p, int shift, int phase, float* wt, float scale = 1.0f) {
  const uint32_t one = 1u << shift, half = one >> 1;
  const int f = (int)(p & (one - 1u));
  const float inv = 1.0f / (float)one;
  if constexpr (ASSIGN == CNPC_TSC) {
    int off, dfix;
    if (phase == 0) {
      const bool up = f >= (int)half;
      off = up ? 1 : 0;
      dfix = up ? f - (int)one : f;
    } else {
      off = 0;
      dfix = f - (int)half;
    }
    const float d = (float)dfix * inv;
    const float a = 0.5f - d, b = 0.5f + d;
    wt[0] = (0.5f * scale) * a * a;
    wt[1] = __builtin_fmaf(-d, d * scale, 0.75f * scale);
    wt[2] = (0.5f * scale) * b * b;
    return off - 1;
  } else {
    if (phase == 0) {
      const float d = (float)f * inv;
      wt[0] = __builtin_fmaf(-d, scale, scale);
      wt[1] = d * scale;
      return 0;
    }
    const bool up = f >= (int)half;
    const int off = up ? 0 : -1;
    const int dfix = up ? f - (int)half : f + (int)half;
    const float d = (float)dfix * inv;
    wt[0] = __builtin_fmaf(-d, scale, scale);
    wt[1] = d * scale;
    return off;
  }
}

template <int ASSIGN>
__global__ void __launch_bounds__(PAINT32_THREADS, 8) k_paint_tiles_u32(PaintCats<float, 3> pc, TileGeom g, int nphase,
                                                                     bool packed) {
  const Rec<3>* __restrict__ rec = pc.rec[blockIdx.y];
  const uint32_t* __restrict__ start = pc.start[blockIdx.y];
  const uint32_t* __restrict__ count = pc.count[blockIdx.y];
  float* __restrict__ blocks = pc.blocks[blockIdx.y];
  constexpr float SCALE = 2097152.0f;  // 2^21
  constexpr int ROUNDS_PER_FLUSH = ASSIGN == CNPC_TSC ? 4 : 1;
  constexpr int NP = ASSIGN == CNPC_TSC ? 3 : 2;
  __shared__ __align__(16) uint32_t acc[2 * BVOL];
  const int t = blockIdx.x;
  const int shift = g.shift;
  const int nv = nphase * BVOL;
  for (int i = threadIdx.x; i < nv; i += PAINT32_THREADS) acc[i] = 0u;
  unsigned long long own[PAINT32_OWN];
#pragma unroll
  for (int j = 0; j < PAINT32_OWN; ++j) own[j] = 0ull;
  __syncthreads();
  const int key = key_of(t / (g.nt * g.nt), (t / g.nt) % g.nt, t % g.nt, g);
  const uint32_t s0 = start[key], cnt = count[key];
  int round = 0;
  for (uint32_t base = 0; base < cnt; base += PAINT32_THREADS) {
    const uint32_t k = base + threadIdx.x;
    if (k < cnt) {
      uint32_t px, py, pz;
      if (packed) {  // pack_rec: tile-relative positions on the 2^-17 cell grid
        const uint64_t q = reinterpret_cast<const uint64_t*>(rec)[(int64_t)s0 + k];
        const int up = shift - 17;
        px = (uint32_t)(q & 0x1fffffu) << up;
        py = (uint32_t)((q >> 21) & 0x1fffffu) << up;
        pz = (uint32_t)((q >> 42) & 0x1fffffu) << up;
      } else {
        const Rec<3> p = rec[(int64_t)s0 + k];
        px = p.v[0];
        py = p.v[1];
        pz = p.v[2];
      }
      const int bx = ((int)(px >> shift) & 15) + 1;
      const int by = ((int)(py >> shift) & 15) + 1;
      const int bz = ((int)(pz >> shift) & 15) + 1;
      for (int ph = 0; ph < nphase; ++ph) {
        float wx[3], wy[3], wz[3];
        const int ox = stencil32<ASSIGN>(px, shift, ph, wx, SCALE);  // x weights carry the 2^21 units
        const int oy = stencil32<ASSIGN>(py, shift, ph, wy);
        const int oz = stencil32<ASSIGN>(pz, shift, ph, wz);
        // node lz = bz + oz + iz sits at lz - 1 in its row, lz = 0 at 18
        const int a1 = ph * BVOL + (bx + ox) * BW * BW + (by + oy) * BW + (bz + oz - 1);
        const int a0 = a1 + (bz + oz == 0 ? BW : 0);
#pragma unroll
        for (int ix = 0; ix < NP; ++ix)
#pragma unroll
          for (int iy = 0; iy < NP; ++iy) {
            const float vxy = wx[ix] * wy[iy];
            const int o = ix * BW * BW + iy * BW;
#pragma unroll
            for (int iz = 0; iz < NP; ++iz)
              atomicAdd(&acc[(iz == 0 ? a0 : a1) + o + iz], (uint32_t)__builtin_fmaf(vxy, wz[iz], 0.5f));
          }
      }
    }
    if (++round == ROUNDS_PER_FLUSH || base + PAINT32_THREADS >= cnt) {
      round = 0;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < PAINT32_OWN; ++j) {
        const int i = threadIdx.x + j * PAINT32_THREADS;
        if (i < nv) {
          own[j] += acc[i];
          acc[i] = 0u;
        }
      }
      __syncthreads();
    }
  }
  float* out = blocks + (int64_t)t * nphase * BSTRIDE;
#pragma unroll
  for (int j = 0; j < PAINT32_OWN; ++j) {
    const int i = threadIdx.x + j * PAINT32_THREADS;
    if (i < nv) {
      const int q = i >= BVOL ? 1 : 0;
      out[q * BSTRIDE + i - q * BVOL] = (float)((double)own[j] * (1.0 / (double)SCALE));
    }
  }
}

// 16 consecutive elements from an address aligned to the element size
// (gfx950 takes 16-byte loads at 4-byte alignment)
template <typename T>
__device__ __forceinline__ void load16(const T* __restrict__ p, T* v) {
  struct __attribute__((aligned(sizeof(T)))) V2 { T a, b; };
  struct __attribute__((aligned(sizeof(T)))) V4 { T a, b, c, d; };
  if constexpr (sizeof(T) == 4) {
    const V4* q = reinterpret_cast<const V4*>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const V4 u = q[k];
      v[4 * k] = u.a; v[4 * k + 1] = u.b; v[4 * k + 2] = u.c; v[4 * k + 3] = u.d;
    }
  } else {
    const V2* q = reinterpret_cast<const V2*>(p);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const V2 u = q[k];
      v[2 * k] = u.a; v[2 * k + 1] = u.b;
    }
  }
}

// 16 consecutive elements to a 16 * sizeof(T)-aligned address
template <typename T>
__device__ __forceinline__ void store16(T* __restrict__ p, const T* v) {
  if constexpr (sizeof(T) == 4) {
    float4* q = reinterpret_cast<float4*>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
  } else {
    double2* q = reinterpret_cast<double2*>(p);
#pragma unroll
    for (int k = 0; k < 8; ++k) q[k] = make_double2(v[2 * k], v[2 * k + 1]);
  }
}

// Fold of the tile blocks into meshes.  A workgroup covers Z2 tiles along z
// of one (x, y) tile column and one phase; a thread owns the 16-node z-row
// (x, y) of one tile.  Along x (and y) the row gathers from its own tile
// (local row l = c + 1) and, for c = 0, 1 (15), from the lower neighbour's
// row l = c + 17 (the upper neighbour's row 0); from each of these <= 4 (x, y)
// sources it reads the 16 own values of the row in the same z tile, values
// 16..17 of the row in the lower z tile (nodes 0, 1) and value 18 of the row
// in the upper z tile (node 15): every block element is read exactly once.
// Per set the sum is formed first, then delta = sum_s cd[s] v_s and
// N = sum_s cn[s] v_s.
template <typename T>
__global__ void __launch_bounds__(512) k_fold_tiles(FoldArgs<T> fa, const double* __restrict__ norms,
                                                    T* __restrict__ delta, T* __restrict__ noise) {
  const int n = fa.n, nt = fa.nt, z2 = nt >= 2 ? 2 : 1;
  const int nzp = nt / z2;
  const int rows = blockDim.x / z2, parts = 256 / rows;  // rows of a tile per workgroup
  // workgroups go to the 8 XCDs in turn (launch index mod 8); give each XCD a
  // contiguous range of tile columns so that the halo rows shared by
  // neighbouring tiles are fetched into one L2 (a bijection when 8 | grid)
  int b = blockIdx.x;
  if ((gridDim.x & 7u) == 0) b = (int)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3));
  const int part = b % parts; b /= parts;
  const int tzp = b % nzp; b /= nzp;
  const int ty = b % nt; b /= nt;
  const int tx = b % nt;
  const int ph = b / nt;
  const int zt = threadIdx.x % z2, row = part * rows + threadIdx.x / z2;
  const int cx = row >> 4, cy = row & 15;
  const int tz = tzp * z2 + zt;
  const double alpha = norms[CNPC_NORM_ALPHA];
  T cd[4] = {T(0), T(0), T(0), T(0)}, cn[4] = {T(0), T(0), T(0), T(0)};
  if (fa.nsets == 2) {
    cd[0] = T(1); cd[1] = T(-alpha); cn[0] = T(1); cn[1] = T(alpha * alpha);
  } else {
    cd[0] = T(1); cd[1] = T(-alpha); cn[2] = T(1); cn[3] = T(alpha * alpha);
  }
  // x / y sources: own tile (row c + 1) or, near the faces, the neighbour
  const bool hx = cx <= 1 || cx == 15, hy = cy <= 1 || cy == 15;
  const int txn = cx <= 1 ? (tx - 1 + nt) % nt : (tx + 1) % nt;
  const int tyn = cy <= 1 ? (ty - 1 + nt) % nt : (ty + 1) % nt;
  const int lxn = cx <= 1 ? cx + 17 : 0, lyn = cy <= 1 ? cy + 17 : 0;
  const int tzl = (tz - 1 + nt) % nt, tzu = (tz + 1) % nt;
  const int64_t bst = (int64_t)fa.nphase * BSTRIDE;  // per tile
  // element offsets of the row of source k = 2 a + c (a: x neighbour, c: y
  // neighbour) in the same, lower and upper z tile; source k is used when ok[k]
  int64_t o0[4], o1[4], o2[4];
  bool ok[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int a = k >> 1, c = k & 1;
    ok[k] = (!a || hx) && (!c || hy);
    const int txs = a ? txn : tx, tys = c ? tyn : ty;
    const int r = ((a ? lxn : cx + 1) * BW + (c ? lyn : cy + 1)) * BW;
    const int64_t col = ((int64_t)txs * nt + tys) * nt;
    o0[k] = (col + tz) * bst + (int64_t)ph * BSTRIDE + r;
    o1[k] = (col + tzl) * bst + (int64_t)ph * BSTRIDE + r + 16;
    o2[k] = (col + tzu) * bst + (int64_t)ph * BSTRIDE + r + 18;
  }
  T d[16], q[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) d[e] = q[e] = T(0);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s >= fa.nsets) break;
    const T* __restrict__ bl = fa.blocks[s];
    T v[16];
    load16<T>(bl + o0[0], v);
    T lo0 = bl[o1[0]], lo1 = bl[o1[0] + 1], up = bl[o2[0]];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      if (!ok[k]) continue;
      T u[16];
      load16<T>(bl + o0[k], u);
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] += u[e];
      lo0 += bl[o1[k]];
      lo1 += bl[o1[k] + 1];
      up += bl[o2[k]];
    }
    v[0] += lo0;
    v[1] += lo1;
    v[15] += up;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      d[e] += cd[s] * v[e];
      q[e] += cn[s] * v[e];
    }
  }
  const int64_t idx = (int64_t)ph * n * n * n + ((int64_t)(tx * 16 + cx) * n + ty * 16 + cy) * n + tz * 16;
  store16<T>(delta + idx, d);
  if (noise) store16<T>(noise + idx, q);
}

// Fold for meshes of 256 and 512: a workgroup takes RW = 256 / nt rows (x, y) of a
// tile column, one lane per row and z tile (lane (cy, tz): 16 lanes read rows that
// are consecutive in a block), so that the z halos stay inside the workgroup:
// summed rows are staged in LDS, the halo values added there after a barrier (one
// writer per node), and whole mesh rows stored.  A lane without a y halo reads its
// own row for the y-neighbour sources and weighs them by zero, so that no load
// sits in a divergent branch.  Same sums as k_fold_tiles up to rounding.  Bound by
// HBM: 512^3 FP32, both meshes, 5.8 GB, 1530 us with a tile pair's rows per workgroup
// (k_fold_tiles) before, 1199 here (4.8 TB/s); 512^3 FP64 one mesh 3161 before, 2557
// here; 256^3 FP64 one mesh 328 before, 275 here, both 428 before, 328 here.
template <typename T, int NT_>
__global__ void __launch_bounds__(256) k_fold_rows(FoldArgs<T> fa, const double* __restrict__ norms,
                                                   T* __restrict__ delta, T* __restrict__ noise) {
  constexpr int N = 16 * NT_, RW = 256 / NT_;  // nodes per row, rows per workgroup
  static_assert(RW <= 16, "rows of one x node");
  constexpr int RS = N + NT_;                  // staged row stride (one of padding per 16)
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* stage = reinterpret_cast<cx<T>*>(smem_raw);  // [RW][RS]
  // workgroups go to the 8 XCDs in turn: each XCD takes a contiguous range of
  // tile columns, so the blocks and halo rows they share meet in one L2
  int b = (int)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3));
  const int row0 = (b % (256 / RW)) * RW;
  b /= 256 / RW;
  const int ty = b % NT_;
  b /= NT_;
  const int tx = b % NT_;
  const int ph = b / NT_;
  const int tz = threadIdx.x / RW, lr = threadIdx.x % RW;
  const int c_x = (row0 + lr) >> 4, cy = (row0 + lr) & 15;
  const double alpha = norms[CNPC_NORM_ALPHA];
  T cd[4] = {T(0), T(0), T(0), T(0)}, cn[4] = {T(0), T(0), T(0), T(0)};
  if (fa.nsets == 2) {
    cd[0] = T(1); cd[1] = T(-alpha); cn[0] = T(1); cn[1] = T(alpha * alpha);
  } else {
    cd[0] = T(1); cd[1] = T(-alpha); cn[2] = T(1); cn[3] = T(alpha * alpha);
  }
  // the workgroup's RW <= 16 rows share x node c_x: hx is uniform
  const bool hx = c_x <= 1 || c_x == 15, hy = cy <= 1 || cy == 15;
  const int txn = c_x <= 1 ? (tx - 1 + NT_) % NT_ : (tx + 1) % NT_;
  const int tyn = cy <= 1 ? (ty - 1 + NT_) % NT_ : (ty + 1) % NT_;
  const int lxn = c_x <= 1 ? c_x + 17 : 0, lyn = cy <= 1 ? cy + 17 : 0;
  const int64_t bst = (int64_t)fa.nphase * BSTRIDE;
  int64_t o[4];  // source k = 2 a + c (a: x neighbour, c: y neighbour)
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const bool a = k >> 1, c = (k & 1) && hy;
    o[k] = (((int64_t)(a ? txn : tx) * NT_ + (c ? tyn : ty)) * NT_ + tz) * bst + (int64_t)ph * BSTRIDE +
           ((a ? lxn : c_x + 1) * BW + (c ? lyn : cy + 1)) * BW;
  }
  const T fy = hy ? T(1) : T(0);
  T d[19], q[19];
#pragma unroll
  for (int e = 0; e < 19; ++e) d[e] = q[e] = T(0);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s >= fa.nsets) break;
    const T* __restrict__ bl = fa.blocks[s];
    T v[19], u[19];
    load16<T>(bl + o[0], v);
    v[16] = bl[o[0] + 16]; v[17] = bl[o[0] + 17]; v[18] = bl[o[0] + 18];
    load16<T>(bl + o[1], u);
    u[16] = bl[o[1] + 16]; u[17] = bl[o[1] + 17]; u[18] = bl[o[1] + 18];
#pragma unroll
    for (int e = 0; e < 19; ++e) v[e] += fy * u[e];
    if (hx) {
      load16<T>(bl + o[2], u);
      u[16] = bl[o[2] + 16]; u[17] = bl[o[2] + 17]; u[18] = bl[o[2] + 18];
#pragma unroll
      for (int e = 0; e < 19; ++e) v[e] += u[e];
      load16<T>(bl + o[3], u);
      u[16] = bl[o[3] + 16]; u[17] = bl[o[3] + 17]; u[18] = bl[o[3] + 18];
#pragma unroll
      for (int e = 0; e < 19; ++e) v[e] += fy * u[e];
    }
#pragma unroll
    for (int e = 0; e < 19; ++e) {
      d[e] += cd[s] * v[e];
      q[e] += cn[s] * v[e];
    }
  }
  // staged node (row, z) at row * RS + z + z / 16
  cx<T>* srow = stage + lr * RS;
#pragma unroll
  for (int e = 0; e < 16; ++e) srow[17 * tz + e] = cx<T>{d[e], q[e]};
  __syncthreads();
  {
    cx<T>* up = srow + 17 * ((tz + 1) % NT_);
    cx<T>* lo = srow + 17 * ((tz + NT_ - 1) % NT_) + 15;
    up[0] = cadd(up[0], cx<T>{d[16], q[16]});
    up[1] = cadd(up[1], cx<T>{d[17], q[17]});
    *lo = cadd(*lo, cx<T>{d[18], q[18]});
  }
  __syncthreads();
  for (int i = threadIdx.x; i < RW * N; i += 256) {
    const int r = i / N, z = i % N, gr = row0 + r;
    const cx<T> v = stage[r * RS + z + (z >> 4)];
    const int64_t idx = (((int64_t)ph * N + 16 * tx + (gr >> 4)) * N + 16 * ty + (gr & 15)) * N + z;
    delta[idx] = v.x;
    if (noise) noise[idx] = v.y;
  }
}

// Fold fused with the z pass of the de-interlacing transforms (N = 256: 16
// z-tiles, one z-row = one row_fft_rr of 16 lanes).  A workgroup takes the 16
// node rows (x, y = 16 ty + cy) of one x node x = 16 tx + cx of the tile
// column (ph, tx, ty).  Load phase, lane (cy, tz): the block rows that hold
// the 16 nodes of z-tile tz of row cy (own tile, the x / y neighbours' halo
// rows; rows of consecutive cy are contiguous in a block, so 16 lanes read
// 16 x 19 consecutive elements) are summed over the sources, and over both
// weight sets into delta = sum cd v and N = sum cn v, then staged in LDS; the
// row's z halo (positions 16, 17: nodes 0, 1 of z-tile tz + 1; position 18:
// node 15 of z-tile tz - 1) is added after a barrier, one writer per node.
// Transform phase: group g transforms row g (delta + i N) and the two-for-one
// split gives the r2c z transforms of delta (kz < kz_d) and N (kz < kz_n).
// Sources that a lane does not need are read from its own row and weighted by
// zero, so no load sits in a divergent branch.  The meshes are never written.
constexpr int FZ_RS = 273;  // staged row stride (complex): 256 nodes + 1 pad per 16

template <typename T>
__global__ void __launch_bounds__(256) k_fold_zr2c(FoldArgs<T> fa, const double* __restrict__ norms,
                                                   cx<T>* __restrict__ dsp, int kz_d, cx<T>* __restrict__ nw1,
                                                   int kz_n) {
  constexpr int R = 16, N = 256;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<T>* tw = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* stage = tw + N;  // [16][FZ_RS]; later the row_fft_rr buffers
  load_twiddles<T, N, -1>(tw);
  // workgroups go to the 8 XCDs in turn: each XCD takes a contiguous range of
  // tile columns, so the blocks and halo rows they share meet in one L2
  int b = blockIdx.x;
  if ((gridDim.x & 7u) == 0) b = (int)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3));
  const int nt = fa.nt;
  const int cx_ = b & 15;
  b >>= 4;
  const int ty = b % nt;
  b /= nt;
  const int tx = b % nt;
  const int ph = b / nt;
  const int tz = threadIdx.x >> 4, cy = threadIdx.x & 15;
  const double alpha = norms[CNPC_NORM_ALPHA];
  T cd[4] = {T(0), T(0), T(0), T(0)}, cn[4] = {T(0), T(0), T(0), T(0)};
  if (fa.nsets == 2) {
    cd[0] = T(1); cd[1] = T(-alpha); cn[0] = T(1); cn[1] = T(alpha * alpha);
  } else {
    cd[0] = T(1); cd[1] = T(-alpha); cn[2] = T(1); cn[3] = T(alpha * alpha);
  }
  // hx is uniform over the workgroup; a lane without a y halo reads its own
  // row for the y-neighbour sources and weighs them by fy = 0
  const bool hx = cx_ <= 1 || cx_ == 15, hy = cy <= 1 || cy == 15;
  const int txn = cx_ <= 1 ? (tx - 1 + nt) % nt : (tx + 1) % nt;
  const int tyn = cy <= 1 ? (ty - 1 + nt) % nt : (ty + 1) % nt;
  const int lxn = cx_ <= 1 ? cx_ + 17 : 0, lyn = cy <= 1 ? cy + 17 : 0;
  const int64_t bst = (int64_t)fa.nphase * BSTRIDE;
  int64_t o[4];  // source k = 2 a + c (a: x neighbour, c: y neighbour)
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int a = k >> 1;
    const bool c = (k & 1) && hy;
    const int txs = a ? txn : tx, tys = c ? tyn : ty;
    const int r = ((a ? lxn : cx_ + 1) * BW + (c ? lyn : cy + 1)) * BW;
    o[k] = (((int64_t)txs * nt + tys) * nt + tz) * bst + (int64_t)ph * BSTRIDE + r;
  }
  const T fy = hy ? T(1) : T(0);
  T d[19], q[19];
#pragma unroll
  for (int e = 0; e < 19; ++e) d[e] = q[e] = T(0);
#pragma unroll
  for (int sidx = 0; sidx < 4; ++sidx) {
    if (sidx >= fa.nsets) break;
    const T* __restrict__ bl = fa.blocks[sidx];
    T v[19], u[19];
    load16<T>(bl + o[0], v);
    v[16] = bl[o[0] + 16]; v[17] = bl[o[0] + 17]; v[18] = bl[o[0] + 18];
    load16<T>(bl + o[1], u);
    u[16] = bl[o[1] + 16]; u[17] = bl[o[1] + 17]; u[18] = bl[o[1] + 18];
#pragma unroll
    for (int e = 0; e < 19; ++e) v[e] += fy * u[e];
    if (hx) {
      load16<T>(bl + o[2], u);
      u[16] = bl[o[2] + 16]; u[17] = bl[o[2] + 17]; u[18] = bl[o[2] + 18];
#pragma unroll
      for (int e = 0; e < 19; ++e) v[e] += u[e];
      load16<T>(bl + o[3], u);
      u[16] = bl[o[3] + 16]; u[17] = bl[o[3] + 17]; u[18] = bl[o[3] + 18];
#pragma unroll
      for (int e = 0; e < 19; ++e) v[e] += fy * u[e];
    }
#pragma unroll
    for (int e = 0; e < 19; ++e) {
      d[e] += cd[sidx] * v[e];
      q[e] += cn[sidx] * v[e];
    }
  }
  // staged node (row, z) at row * FZ_RS + z + z / 16
  cx<T>* srow = stage + cy * FZ_RS;
#pragma unroll
  for (int e = 0; e < 16; ++e) srow[17 * tz + e] = cx<T>{d[e], q[e]};
  __syncthreads();
  {
    cx<T>* up = srow + 17 * ((tz + 1) & 15);
    cx<T>* lo = srow + 17 * ((tz + 15) & 15) + 15;
    up[0] = cadd(up[0], cx<T>{d[16], q[16]});
    up[1] = cadd(up[1], cx<T>{d[17], q[17]});
    *lo = cadd(*lo, cx<T>{d[18], q[18]});
  }
  __syncthreads();
  const int grp = threadIdx.x >> 4, rank = threadIdx.x & 15;
  cx<T> v[R];
#pragma unroll
  for (int n2 = 0; n2 < R; ++n2) v[n2] = stage[grp * FZ_RS + 17 * n2 + rank];
  __syncthreads();
  row_fft_rr<T, R, -1>(v, rank, stage + grp * (R * (R + 1)), tw);
  const int src = (R - rank) & (R - 1);
  const int kzmax = kz_d > kz_n ? kz_d : kz_n;
  const int K2 = (kzmax + R - 1) / R;
  const int64_t row = ((int64_t)ph * N + 16 * tx + cx_) * N + 16 * ty + grp;
  cx<T>* od = dsp + row * kz_d;
  cx<T>* on = nw1 + row * kz_n;
#pragma unroll
  for (int k2 = 0; k2 < R / 2; ++k2) {
    if (k2 < K2) {
      const cx<T> a = v[R - 1 - k2];
      const cx<T> sh = {__shfl(a.x, src, R), __shfl(a.y, src, R)};
      const cx<T> zm = cconj(rank ? sh : v[(R - k2) & (R - 1)]);
      const cx<T> zk = v[k2];
      const int k = rank + R * k2;
      const cx<T> dd = csub(zk, zm);
      if (k < kz_d) od[k] = cscale(cadd(zk, zm), T(0.5));
      if (k < kz_n) on[k] = cx<T>{T(0.5) * dd.y, T(-0.5) * dd.x};
    }
  }
}

// ------------------------------------------------------------------- host --
static TileGeom tile_geom(const cnpc_mesh_desc* d);

// workgroups of a sums pass over n particles
static int sums_blocks(int64_t n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(SUMS_BLOCKS, (n + SUMS_THREADS - 1) / SUMS_THREADS));
}

static cnpc_status sums_counted(const cnpc_mesh_desc* d, const uint32_t* pos, const float* w, int64_t n,
                                int lmax, double* sums, double* partial, const CountArgs& ca, hipStream_t s) {
  const int nblocks = sums_blocks(n);
  SumsArgs a;
  a.lmax = lmax;
  a.boxsize = d->boxsize;
  for (int i = 0; i < 3; ++i) { a.obs[i] = d->observer[i]; a.los[i] = d->los[i]; }
  a.global_los = d->los_mode == CNPC_LOS_GLOBAL;
  const size_t lds = (ca.count && ca.ntiles <= LDS_TILES_MAX) ? (size_t)ca.ntiles * 4 : 0;
  kt_begin(CNPC_KT_SUMS, s);
  if (lmax >= 4)
    hipLaunchKernelGGL(k_catalog_sums<4>, dim3(nblocks), dim3(SUMS_THREADS), lds, s, pos, w, n, a, partial, ca);
  else if (lmax >= 2)
    hipLaunchKernelGGL(k_catalog_sums<2>, dim3(nblocks), dim3(SUMS_THREADS), lds, s, pos, w, n, a, partial, ca);
  else
    hipLaunchKernelGGL(k_catalog_sums<0>, dim3(nblocks), dim3(SUMS_THREADS), lds, s, pos, w, n, a, partial, ca);
  kt_end(CNPC_KT_SUMS, s);
  CNPC_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_reduce_partials, dim3(CNPC_SUMS_LEN), dim3(64), 0, s, partial, nblocks, sums);
  CNPC_HIP(hipGetLastError());
  return CNPC_OK;
}

cnpc_status launch_catalog_sums(const cnpc_mesh_desc* d, const uint32_t* pos, const float* w,
                                int64_t n, double* sums, void* ws, size_t ws_bytes,
                                hipStream_t s) {
  const int nblocks = SUMS_BLOCKS;
  if (ws_bytes < (size_t)nblocks * CNPC_SUMS_LEN * sizeof(double)) {
    set_error("catalog_sums workspace too small");
    return CNPC_EWORKSPACE;
  }
  CountArgs ca;
  ca.ntiles = 0;
  ca.count = nullptr;
  return sums_counted(d, pos, w, n, 4, sums, reinterpret_cast<double*>(ws), ca, s);
}

cnpc_status launch_norms(const cnpc_mesh_desc* d, const double* gs, const double* rs, int64_t ngal,
                         double* norms, hipStream_t s) {
  hipLaunchKernelGGL(k_norms, dim3(1), dim3(64), 0, s, gs, rs, ngal, d->boxsize, norms);
  CNPC_HIP(hipGetLastError());
  return CNPC_OK;
}

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

static TileGeom tile_geom(const cnpc_mesh_desc* d) {
  TileGeom g;
  g.shift = 32 - ilog2_host(d->n);
  g.nt = d->n / TILE;
  const int S = g.nt < 4 ? g.nt : 4;
  g.ls = ilog2_host(S);
  g.lnb = ilog2_host(g.nt / S);
  return g;
}

// Bucket-pass geometry: chunk of BUCKET_NT * per particles (per <= 8), at most
// BUCKET_BLOCKS_MAX persistent workgroups; a bucket region holds 1.5 times the
// mean bucket count plus the largest chunk (more goes to the overflow region).
constexpr int BUCKET_NT = 1024;
constexpr int BUCKET_BLOCKS_MAX = 512;
constexpr int OVF_BLOCKS = 256;  // workgroups walking the overflow records: 512 cost a batch 0.3%
static uint32_t bucket_cap(int64_t n, int nbuckets) {
  const int64_t mean = (n + nbuckets - 1) / nbuckets;
  const int64_t c = mean + mean / 2 + (int64_t)BUCKET_NT * 8;
  return (uint32_t)((c + 63) / 64 * 64);
}

PaintLayout paint_layout(const cnpc_mesh_desc* d, int64_t ngal, int64_t nran, bool weighted) {
  PaintLayout L;
  const int nt = d->n / TILE;
  L.nt = nt;
  L.ntiles = nt * nt * nt;
  L.nphase = d->interlace ? 2 : 1;
  L.nsets = weighted ? 4 : 2;
  const TileGeom g = tile_geom(d);
  L.nbuckets = 1 << (3 * g.lnb);
  const size_t es = esize(d->dtype);
  const int64_t np = ngal > nran ? ngal : nran;
  const size_t rec = (size_t)np * (weighted ? 16 : 12);
  size_t off = 0;
  // a mesh of one bucket sorts both catalogs at once (paint_small)
  L.off_rec = off; off = align_up(off + rec);
  if (L.nbuckets == 1) off = align_up(off + rec);
  L.off_tmp = off; off = align_up(off + (L.nbuckets > 1 ? rec : 0));
  L.off_count[0] = off; off = align_up(off + (size_t)L.ntiles * 4);
  L.off_count[1] = off; off = align_up(off + (size_t)L.ntiles * 4);
  L.off_partial = off; off = align_up(off + (size_t)BUCKET_BLOCKS_MAX * CNPC_SUMS_LEN * 8);
  L.off_sums = off; off = align_up(off + (size_t)2 * CNPC_SUMS_LEN * 8);
  L.off_start = off; off = align_up(off + (L.nbuckets == 1 ? 2 * SMALL_TILES : (size_t)L.ntiles) * 4);
  L.off_cursor = off; off = align_up(off + (size_t)L.ntiles * 4);
  L.off_hist = off; off = align_up(off + (L.nbuckets == 1 ? (size_t)2 * SUMS_BLOCKS * SMALL_TILES * 4 : 0));
  L.off_bcur = off; off = align_up(off + (size_t)L.nbuckets * 4);
  for (int k = 0; k < L.nsets; ++k) {
    L.off_blocks[k] = off;
    off = align_up(off + (size_t)L.ntiles * L.nphase * BSTRIDE * es);
  }
  L.cap = 0;
  L.off_region = L.off_ovf = L.off_bcnt = off;
  if (L.nbuckets > 1) {
    const size_t rs = weighted ? 16 : 12;
    L.cap = bucket_cap(np, L.nbuckets);
    L.off_region = off; off = align_up(off + (size_t)L.nbuckets * L.cap * rs);
    L.off_ovf = off; off = align_up(off + (size_t)np * rs);
    L.off_bcnt = off; off = align_up(off + (size_t)(L.nbuckets + 1) * 4);
  }
  L.total = off;
  return L;
}

__global__ void k_zero_u32(uint32_t* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

constexpr int FINE_RCAP = 512;  // LDS key range of the second sort step

// Particles per thread for nt-thread workgroups: the tuned value when its LDS
// layout fits, else the largest (4, 2, 1) whose layout lets 32 waves' worth
// of workgroups share a CU, else the largest that fits one.
static int partition_per(int rs, int rcap, int nt) {
  const size_t lim = lds_limit();
  const int tp = tune_value(CNPC_TUNE_SORT_PER);
  if (tp > 0 && partition_lds(tp, rs, rcap, nt) <= lim) return tp;
  const size_t wgs = (size_t)(2048 / nt);
  for (int per = 4; per >= 1; per >>= 1)
    if (wgs * partition_lds(per, rs, rcap, nt) <= lim) return per;
  for (int per = 4; per >= 1; per >>= 1)
    if (partition_lds(per, rs, rcap, nt) <= lim) return per;
  return 0;
}

template <bool FINE, int RS, int NT>
static void launch_partition_nt(int per, unsigned nblk, size_t lds, const uint32_t* pos, const float* w,
                                const Rec<RS>* rin, int64_t n, const TileGeom& g, int rcap, uint32_t* cursor,
                                Rec<RS>* rout, bool pack, hipStream_t s) {
  if (per == 4)
    hipLaunchKernelGGL((k_partition<FINE, RS, 4, NT>), dim3(nblk), dim3(NT), lds, s, pos, w, rin, n, g,
                       rcap, cursor, rout, pack);
  else if (per == 2)
    hipLaunchKernelGGL((k_partition<FINE, RS, 2, NT>), dim3(nblk), dim3(NT), lds, s, pos, w, rin, n, g,
                       rcap, cursor, rout, pack);
  else
    hipLaunchKernelGGL((k_partition<FINE, RS, 1, NT>), dim3(nblk), dim3(NT), lds, s, pos, w, rin, n, g,
                       rcap, cursor, rout, pack);
}

template <bool FINE, int RS>
static cnpc_status launch_partition(const uint32_t* pos, const float* w, const Rec<RS>* rin, int64_t n,
                                    const TileGeom& g, int rcap, uint32_t* cursor, Rec<RS>* rout, bool pack,
                                    hipStream_t s) {
  const int nt = tune_value(CNPC_TUNE_SORT_THREADS) == 512 ? 512 : 1024;
  const int per = partition_per(RS, rcap, nt);
  if (per == 0) {
    set_error("sort: %d keys do not fit the LDS of a workgroup", rcap);
    return CNPC_EINVAL;
  }
  const int64_t ch = (int64_t)nt * per;
  const unsigned nblk = (unsigned)((n + ch - 1) / ch);
  const size_t lds = partition_lds(per, RS, rcap, nt);
  kt_begin(CNPC_KT_SORT, s);
  if (nt == 512)
    launch_partition_nt<FINE, RS, 512>(per, nblk, lds, pos, w, rin, n, g, rcap, cursor, rout, pack, s);
  else
    launch_partition_nt<FINE, RS, 1024>(per, nblk, lds, pos, w, rin, n, g, rcap, cursor, rout, pack, s);
  kt_end(CNPC_KT_SORT, s);
  CNPC_HIP(hipGetLastError());
  return CNPC_OK;
}

// Tile painting of tile-sorted records: ncat catalogs in one launch, the w^2 blocks
// with `second`
template <typename T, int RS>
static cnpc_status launch_paint_tiles(const cnpc_mesh_desc* d, bool second, int ncat, const PaintCats<T, RS>& pc,
                                      const PaintLayout& L, hipStream_t s) {
  const TileGeom g = tile_geom(d);
  kt_begin(CNPC_KT_PAINT, s);
  if constexpr (sizeof(T) == 4 && RS == 3) {
    // unit weights: w^2 = w, the second power's blocks are painted alike (with the other
    // catalog's weights in cnpc_paint_deinterlace)
    for (int pw = 0; pw < (second ? 2 : 1); ++pw) {
      PaintCats<T, RS> p = pc;
      for (int c = 0; c < ncat; ++c) p.blocks[c] = pc.blocks[c + 2 * pw];
      hipLaunchKernelGGL((d->assign == CNPC_TSC ? k_paint_tiles_u32<CNPC_TSC> : k_paint_tiles_u32<CNPC_CIC>),
                         dim3(L.ntiles, (unsigned)ncat), dim3(PAINT32_THREADS), 0, s, p, g, L.nphase,
                         packs_records(true, 3, g.shift));
    }
  } else {
    const int npow = second ? 2 : 1;
    hipLaunchKernelGGL((d->assign == CNPC_TSC ? k_paint_tiles<T, CNPC_TSC, RS> : k_paint_tiles<T, CNPC_CIC, RS>),
                       dim3((unsigned)(L.ntiles * L.nphase * npow), (unsigned)ncat), dim3(1024), 0, s, pc, g, L.nphase,
                       npow);
  }
  kt_end(CNPC_KT_PAINT, s);
  CNPC_HIP(hipGetLastError());
  return CNPC_OK;
}

// the records of set set0 (rec, start of the layout, its count)
template <typename T, int RS>
static cnpc_status paint_sorted(const cnpc_mesh_desc* d, bool second, int set0, unsigned char* ws,
                                const PaintLayout& L, hipStream_t s) {
  PaintCats<T, RS> pc{};
  pc.rec[0] = reinterpret_cast<const Rec<RS>*>(ws + L.off_rec);
  pc.start[0] = reinterpret_cast<const uint32_t*>(ws + L.off_start);
  pc.count[0] = reinterpret_cast<const uint32_t*>(ws + L.off_count[set0]);
  pc.blocks[0] = reinterpret_cast<T*>(ws + L.off_blocks[set0]);
  if (second) pc.blocks[2] = reinterpret_cast<T*>(ws + L.off_blocks[set0 + 2]);
  return launch_paint_tiles<T, RS>(d, second, 1, pc, L, s);
}

// Meshes of one tile bucket (N <= 64), both catalogs with weights or both
// without: sums and tile histograms of both catalogs, their reductions with the
// scan and the norms, the sort and the painting, one launch each (13 launches
// with a catalog at a time).  Such passes are bound by the launches: P_0,2 on 32^3
// 171 us with 31 launches before, 146 with 21; P_0,2,4 on 64^3 225 before, 193.
template <typename T, int RS>
static cnpc_status paint_small(const cnpc_mesh_desc* d, const uint32_t* const* pos, const float* const* w,
                               const int64_t* n, bool second, int lmax, double* const* sums, double* norms,
                               unsigned char* ws, const PaintLayout& L, hipStream_t s) {
  const TileGeom g = tile_geom(d);
  SmallPair sp;
  PaintCats<T, RS> pc{};
  int nblk = 1;
  int64_t nmax = 1;
  const size_t rec = ((size_t)std::max(n[0], n[1]) * RS * 4 + 255) & ~(size_t)255;
  for (int c = 0; c < 2; ++c) {
    SmallCat& k = sp.c[c];
    k.pos = pos[c];
    k.w = w[c];
    k.n = n[c];
    k.nblk = sums_blocks(n[c]);
    k.partial = reinterpret_cast<double*>(ws + L.off_partial) + (size_t)c * SUMS_BLOCKS * CNPC_SUMS_LEN;
    k.hist = reinterpret_cast<uint32_t*>(ws + L.off_hist) + (size_t)c * SUMS_BLOCKS * SMALL_TILES;
    k.count = reinterpret_cast<uint32_t*>(ws + L.off_count[c]);
    k.start = reinterpret_cast<uint32_t*>(ws + L.off_start) + c * SMALL_TILES;
    k.rec = ws + L.off_rec + c * rec;
    k.sums = sums[c];
    pc.rec[c] = reinterpret_cast<const Rec<RS>*>(k.rec);
    pc.start[c] = k.start;
    pc.count[c] = k.count;
    pc.blocks[c] = reinterpret_cast<T*>(ws + L.off_blocks[c]);
    if (second) pc.blocks[c + 2] = reinterpret_cast<T*>(ws + L.off_blocks[c + 2]);
    nblk = std::max(nblk, k.nblk);
    nmax = std::max(nmax, n[c]);
  }
  SumsArgs a;
  a.lmax = lmax;
  a.boxsize = d->boxsize;
  for (int i = 0; i < 3; ++i) { a.obs[i] = d->observer[i]; a.los[i] = d->los[i]; }
  a.global_los = d->los_mode == CNPC_LOS_GLOBAL;
  kt_begin(CNPC_KT_SUMS, s);
  hipLaunchKernelGGL((lmax >= 4 ? k_catalog_sums2<4> : lmax >= 2 ? k_catalog_sums2<2> : k_catalog_sums2<0>),
                     dim3((unsigned)nblk, 2), dim3(SUMS_THREADS), L.ntiles * 4, s, sp, a, g, L.ntiles);
  kt_end(CNPC_KT_SUMS, s);
  CNPC_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_small_scan, dim3(3), dim3(1024), 0, s, sp, L.ntiles, n[0], d->boxsize, norms);
  CNPC_HIP(hipGetLastError());
  // 4 runs at a time where a workgroup has more than one
  const int per = nmax > (int64_t)sums_blocks(nmax) * SUMS_THREADS ? 4 : 1;
  kt_begin(CNPC_KT_SORT, s);
  hipLaunchKernelGGL((per == 4 ? k_partition2<RS, 4> : k_partition2<RS, 1>), dim3((unsigned)nblk, 2), dim3(1024),
                     (size_t)1024 * per * (RS * 4 + 2), s, sp, g, L.ntiles);
  kt_end(CNPC_KT_SORT, s);
  CNPC_HIP(hipGetLastError());
  return launch_paint_tiles<T, RS>(d, second, 2, pc, L, s);
}

// Counting sort with a histogram pass of its own (CNPC_TUNE_SORT_FUSED 1, meshes of
// several buckets), then the tile painting.
template <typename T, int RS>
static cnpc_status sort_and_paint(const cnpc_mesh_desc* d, const uint32_t* pos, const float* w, int64_t n,
                                  int set0, bool second, bool counted, unsigned char* ws,
                                  const PaintLayout& L, hipStream_t s) {
  const TileGeom g = tile_geom(d);
  uint32_t* count = reinterpret_cast<uint32_t*>(ws + L.off_count[set0]);
  uint32_t* start = reinterpret_cast<uint32_t*>(ws + L.off_start);
  uint32_t* cursor = reinterpret_cast<uint32_t*>(ws + L.off_cursor);
  uint32_t* bcur = reinterpret_cast<uint32_t*>(ws + L.off_bcur);
  Rec<RS>* rec = reinterpret_cast<Rec<RS>*>(ws + L.off_rec);
  Rec<RS>* tmp = reinterpret_cast<Rec<RS>*>(ws + L.off_tmp);
  if (!counted) {
    hipLaunchKernelGGL(k_zero_u32, dim3(64), dim3(256), 0, s, count, (int64_t)L.ntiles);
    CNPC_HIP(hipGetLastError());
    const size_t lds_count = L.ntiles <= LDS_TILES_MAX ? (size_t)L.ntiles * 4 : 0;
    const int64_t chunk = (int64_t)SORT_BLOCK * SORT_PER_THREAD;
    const int64_t nblk = (n + chunk - 1) / chunk;
    kt_begin(CNPC_KT_SORT, s);
    hipLaunchKernelGGL(k_tile_count, dim3((unsigned)nblk), dim3(SORT_BLOCK), lds_count, s, pos, n, g, L.ntiles,
                       count);
    kt_end(CNPC_KT_SORT, s);
    CNPC_HIP(hipGetLastError());
  }
  hipLaunchKernelGGL((L.ntiles <= 4096 ? k_tile_scan<1> : k_tile_scan<4>), dim3(1), dim3(1024), 0, s, count,
                     L.ntiles, 3 * g.ls, start, cursor, bcur);
  CNPC_HIP(hipGetLastError());
  const bool pack = packs_records(sizeof(T) == 4, RS, g.shift);  // records of the FP32 painter
  CNPC_TRY((launch_partition<false, RS>(pos, w, nullptr, n, g, L.nbuckets, bcur, tmp, false, s)));
  CNPC_TRY((launch_partition<true, RS>(nullptr, nullptr, tmp, n, g, FINE_RCAP, cursor, rec, pack, s)));
  return paint_sorted<T, RS>(d, second, set0, ws, L, s);
}

// Catalog sums, tile histogram and both sort steps from one read of the
// catalog (fused bucket pass), then the tile painting.  sums: CNPC_SUMS_LEN
// doubles (device).
// Bucket-pass shape: CNPC_TUNE_BUCKET 0 (default) 1024 threads; unweighted
// catalogs 8 particles per thread on at most 256 workgroups (one per CU: 130 KB
// of LDS), fewer per thread where such chunks would fill less than 96 CUs (4 up
// to 7.9e5 particles, 2 up to 2.0e5); weighted catalogs 2 on at most 512.  1:
// 1024 threads, 2 particles, next chunk prefetched; 2: 512 threads, 4
// particles, prefetched; 3: 1024 threads, 4 particles on at most 512
// workgroups (1 to 3: unweighted catalogs).
struct BucketShape {
  int nt, per;
  bool pf;
  int maxblk;  // persistent workgroups at most
};
static BucketShape bucket_shape(int rs, int64_t n) {
  const int v = tune_value(CNPC_TUNE_BUCKET);
  if (rs == 3) {
    if (v == 1) return {1024, 2, true, BUCKET_BLOCKS_MAX};
    if (v == 2) return {512, 4, true, BUCKET_BLOCKS_MAX};
  }
  if (rs == 4 || n <= (int64_t)BUCKET_NT * 2 * 96) return {BUCKET_NT, 2, false, BUCKET_BLOCKS_MAX};
  if (v == 3 || n <= (int64_t)BUCKET_NT * 8 * 96) return {BUCKET_NT, 4, false, BUCKET_BLOCKS_MAX};
  return {BUCKET_NT, 8, false, BUCKET_BLOCKS_MAX / 2};
}

template <int RS>
static void launch_bucket_pass(const BucketShape& b, unsigned nblk, size_t lds, const uint32_t* pos, const float* w,
                               int64_t n, const SumsArgs& sa, const BucketArgs& ba, Rec<RS>* region,
                               Rec<RS>* ovf_out, hipStream_t s) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nblk), dim3(b.nt), lds, s, pos, w, n, sa, ba, region, ovf_out);
  };
  if constexpr (RS == 3) {
    if (b.pf && b.nt == 1024) go(k_bucket_pass<3, 2, 1024, true>);
    else if (b.pf) go(k_bucket_pass<3, 4, 512, true>);
    else if (b.per == 8) go(k_bucket_pass<3, 8, BUCKET_NT, false>);
    else if (b.per == 2) go(k_bucket_pass<3, 2, BUCKET_NT, false>);
    else go(k_bucket_pass<3, 4, BUCKET_NT, false>);
  } else {
    go(k_bucket_pass<4, 2, BUCKET_NT, false>);
  }
}

template <typename T, int RS>
static cnpc_status fused_sort_and_paint(const cnpc_mesh_desc* d, const uint32_t* pos, const float* w, int64_t n,
                                        int set0, bool second, int sums_lmax, double* sums, unsigned char* ws,
                                        const PaintLayout& L, hipStream_t s) {
  const TileGeom g = tile_geom(d);
  uint32_t* count = reinterpret_cast<uint32_t*>(ws + L.off_count[set0]);
  uint32_t* start = reinterpret_cast<uint32_t*>(ws + L.off_start);
  uint32_t* cursor = reinterpret_cast<uint32_t*>(ws + L.off_cursor);
  uint32_t* bcur = reinterpret_cast<uint32_t*>(ws + L.off_bcur);
  uint32_t* bcnt = reinterpret_cast<uint32_t*>(ws + L.off_bcnt);
  Rec<RS>* rec = reinterpret_cast<Rec<RS>*>(ws + L.off_rec);
  Rec<RS>* region = reinterpret_cast<Rec<RS>*>(ws + L.off_region);
  Rec<RS>* ovf_rec = reinterpret_cast<Rec<RS>*>(ws + L.off_ovf);
  double* partial = reinterpret_cast<double*>(ws + L.off_partial);
  const uint32_t cap = bucket_cap(n, L.nbuckets);  // <= L.cap
  const bool split_sums = sums_lmax >= 2;  // Y_lm sums in a read of their own
  BucketShape bs = bucket_shape(RS, n);
  const int ltiles = L.ntiles <= LDS_TILES_MAX ? L.ntiles : 0;
  const bool pack = packs_records(sizeof(T) == 4, RS, g.shift);  // records of the FP32 painter
  const bool packb = pack && L.ntiles <= 65536;                  // bucket records packed too
  auto blds = [&](const BucketShape& b) {
    return bucket_pass_lds(b.per, RS, L.nbuckets, b.nt, ltiles) + (packb ? (size_t)b.nt * b.per * 2 : 0);
  };
  size_t lds = blds(bs);
  if (bs.per == 8 && lds > lds_limit()) {  // many buckets (N >= 1024): 4 per thread
    bs = {BUCKET_NT, 4, false, BUCKET_BLOCKS_MAX};
    lds = blds(bs);
  }
  const int64_t ch = (int64_t)bs.nt * bs.per;
  const unsigned nblk = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + ch - 1) / ch, bs.maxblk));
  if (lds > lds_limit()) {
    set_error("bucket pass: %zu bytes of LDS exceed the workgroup limit", lds);
    return CNPC_EUNSUPPORTED;
  }
  hipLaunchKernelGGL(k_zero2_u32, dim3(64), dim3(256), 0, s, count, (int64_t)L.ntiles, bcnt,
                     (int64_t)L.nbuckets + 1);
  CNPC_HIP(hipGetLastError());
  SumsArgs sa;
  sa.lmax = sums_lmax;
  sa.boxsize = d->boxsize;
  for (int i = 0; i < 3; ++i) { sa.obs[i] = d->observer[i]; sa.los[i] = d->los[i]; }
  sa.global_los = d->los_mode == CNPC_LOS_GLOBAL;
  BucketArgs ba;
  ba.g = g;
  ba.ntiles = L.ntiles;
  ba.nbuckets = L.nbuckets;
  ba.cap = cap;
  ba.bcnt = bcnt;
  ba.ovf = bcnt + L.nbuckets;
  ba.tcount = count;
  ba.partial = partial;
  ba.pack = packb;
  ba.rkey = reinterpret_cast<uint16_t*>(reinterpret_cast<uint64_t*>(region) + (int64_t)L.nbuckets * cap);
  ba.okey = reinterpret_cast<uint16_t*>(reinterpret_cast<uint64_t*>(ovf_rec) + n);
  kt_begin(CNPC_KT_SORT, s);
  launch_bucket_pass<RS>(bs, nblk, lds, pos, w, n, sa, ba, region, ovf_rec, s);
  kt_end(CNPC_KT_SORT, s);
  CNPC_HIP(hipGetLastError());
  const int per_bucket = 1 << (3 * g.ls);
  if (ltiles == 0) {
    const int rcpb = (int)((cap + REGION_CHUNK - 1) / REGION_CHUNK);
    kt_begin(CNPC_KT_SORT, s);
    hipLaunchKernelGGL((k_region_count<RS>), dim3((unsigned)(L.nbuckets * rcpb + OVF_BLOCKS)), dim3(1024),
                       region_count_lds(L.nbuckets, 3 * g.ls), s, region,
                       ba.rkey, ovf_rec, ba.okey, bcnt, bcnt + L.nbuckets, cap, rcpb, L.nbuckets, g, packb, count);
    kt_end(CNPC_KT_SORT, s);
    CNPC_HIP(hipGetLastError());
  }
  if (split_sums) {
    CountArgs none;
    none.ntiles = 0;
    none.count = nullptr;
    CNPC_TRY(sums_counted(d, pos, w, n, sums_lmax, sums, partial, none, s));
    hipLaunchKernelGGL((L.ntiles <= 4096 ? k_tile_scan<1> : k_tile_scan<4>), dim3(1), dim3(1024), 0, s, count,
                     L.ntiles, 3 * g.ls, start, cursor, bcur);
  } else {
    // tile scan and the column sums of the bucket pass's partials in one launch
    hipLaunchKernelGGL((L.ntiles <= 4096 ? k_tile_scan_sums<1> : k_tile_scan_sums<4>), dim3(1 + CNPC_SUMS_LEN),
                       dim3(1024), 0, s, count, L.ntiles, start, cursor, partial, (int)nblk, sums);
  }
  CNPC_HIP(hipGetLastError());
  // tile pass: one workgroup per region chunk; then OVF_BLOCKS over the overflow
  const int tper = partition_per(RS, per_bucket, 1024);
  if (tper == 0) {
    set_error("tile pass: %d keys do not fit the LDS of a workgroup", per_bucket);
    return CNPC_EINVAL;
  }
  const int64_t tch = (int64_t)1024 * tper;
  const int cpb = (int)((cap + tch - 1) / tch);
  kt_begin(CNPC_KT_SORT, s);
  auto steps = [&](auto perc) {
    constexpr int PER = decltype(perc)::value;
    const dim3 tgrid((unsigned)(L.nbuckets * cpb)), ogrid(OVF_BLOCKS);
    if (packb) {
      if constexpr (RS == 3) {
        const size_t plds = (size_t)1024 * PER * 10 + (size_t)3 * per_bucket * 4 + 64;
        hipLaunchKernelGGL((k_tile_pass_packed<PER, 1024>), tgrid, dim3(1024), plds, s,
                           reinterpret_cast<const uint64_t*>(region), ba.rkey, bcnt, cap, cpb, g, cursor,
                           reinterpret_cast<uint64_t*>(rec));
        constexpr int OP = ovf_per(PER, 8);
        hipLaunchKernelGGL((k_overflow_pass<RS, OP, 1024, true>), ogrid, dim3(1024),
                           overflow_lds(OP, 8, 1024, L.nbuckets, 3 * g.ls), s, ovf_rec, ba.okey, bcnt + L.nbuckets,
                           L.nbuckets, g, cursor, rec, pack);
      }
    } else {
      hipLaunchKernelGGL((k_tile_pass<RS, PER, 1024>), tgrid, dim3(1024), partition_lds(PER, RS, per_bucket, 1024), s,
                         region, bcnt, cap, cpb, g, cursor, rec, pack);
      constexpr int OP = ovf_per(PER, RS * 4);
      hipLaunchKernelGGL((k_overflow_pass<RS, OP, 1024, false>), ogrid, dim3(1024),
                         overflow_lds(OP, RS * 4, 1024, L.nbuckets, 3 * g.ls), s, ovf_rec, nullptr, bcnt + L.nbuckets,
                         L.nbuckets, g, cursor, rec, pack);
    }
  };
  if (tper == 4) steps(std::integral_constant<int, 4>());
  else if (tper == 2) steps(std::integral_constant<int, 2>());
  else steps(std::integral_constant<int, 1>());
  kt_end(CNPC_KT_SORT, s);
  CNPC_HIP(hipGetLastError());
  return paint_sorted<T, RS>(d, second, set0, ws, L, s);
}

// sums_lmax >= 0: catalog sums into gs / rs and, with form_norms, the norms, along with
// the sort (paint_small for one bucket, whose catalogs are both weighted or both not;
// else the fused bucket pass); < 0, several buckets: sort_and_paint, counted: its tile
// counts already taken.
template <typename T>
static cnpc_status paint_t(const cnpc_mesh_desc* d, const uint32_t* gpos, const float* gw,
                           int64_t ngal, const uint32_t* rpos, const float* rw, int64_t nran,
                           const double* norms, T* delta, T* noise, unsigned char* ws,
                           const PaintLayout& L, bool counted, hipStream_t s, int sums_lmax = -1,
                           double* gs = nullptr, double* rs = nullptr, bool fold = true, bool form_norms = true) {
  // the w^2 blocks are painted and folded only where an N mesh (or the fused fold)
  // takes them; without weights they are the w blocks
  const bool weighted = (gw != nullptr) || (rw != nullptr), second = weighted && (noise != nullptr || !fold);
  const uint32_t* cpos[2] = {gpos, rpos};
  const float* cw[2] = {gw, rw};
  const int64_t cn[2] = {ngal, nran};
  FoldArgs<T> fa;
  fa.n = d->n;
  fa.nt = L.nt;
  fa.nphase = L.nphase;
  fa.nsets = second ? 4 : 2;
  const bool small = L.nbuckets == 1;
  if (small) {
    double* sums_c[2] = {gs, rs};
    double* nm = form_norms ? const_cast<double*>(norms) : nullptr;
    if (weighted) CNPC_TRY((paint_small<T, 4>(d, cpos, cw, cn, second, sums_lmax, sums_c, nm, ws, L, s)));
    else CNPC_TRY((paint_small<T, 3>(d, cpos, cw, cn, false, sums_lmax, sums_c, nm, ws, L, s)));
  }
  for (int c = 0; c < 2; ++c) {
    for (int pw = 0; pw < (second ? 2 : 1); ++pw)
      fa.blocks[c + 2 * pw] = reinterpret_cast<T*>(ws + L.off_blocks[c + 2 * pw]);
    if (small) continue;
    double* sums_c = c == 0 ? gs : rs;
    if (sums_lmax >= 0 && cw[c])
      CNPC_TRY((fused_sort_and_paint<T, 4>(d, cpos[c], cw[c], cn[c], c, second, sums_lmax, sums_c, ws, L, s)));
    else if (sums_lmax >= 0)
      CNPC_TRY((fused_sort_and_paint<T, 3>(d, cpos[c], nullptr, cn[c], c, second, sums_lmax, sums_c, ws, L, s)));
    else if (cw[c])
      CNPC_TRY((sort_and_paint<T, 4>(d, cpos[c], cw[c], cn[c], c, second, counted, ws, L, s)));
    else
      CNPC_TRY((sort_and_paint<T, 3>(d, cpos[c], nullptr, cn[c], c, second, counted, ws, L, s)));
  }
  if (sums_lmax >= 0 && form_norms && !small) CNPC_TRY(launch_norms(d, gs, rs, ngal, const_cast<double*>(norms), s));
  if (!fold) return CNPC_OK;
  kt_begin(CNPC_KT_FOLD, s);
  auto rows = [&](auto ntc) {
    constexpr int NT_ = decltype(ntc)::value, RW = 256 / NT_;
    const unsigned nb = (unsigned)(L.nphase * NT_ * NT_ * (256 / RW));  // a multiple of 8
    hipLaunchKernelGGL((k_fold_rows<T, NT_>), dim3(nb), dim3(256), sizeof(cx<T>) * RW * 17 * NT_, s, fa, norms, delta,
                       noise);
  };
  // 256, 512: whole rows; smaller meshes keep the z-tile pairs (128^3 FP64 74 us, 89
  // in rows), where more workgroups than rows fill the CUs
  if (L.nt == 16) {
    rows(std::integral_constant<int, 16>());
  } else if (L.nt == 32) {
    rows(std::integral_constant<int, 32>());
  } else {
    const int z2 = L.nt >= 2 ? 2 : 1;
    // a tile pair's 256 rows in one workgroup; on meshes of 64 tiles and less 32 rows
    // (one wavefront), so that more CUs take part (64^3: 14 us in one, 5.9 in eight)
    const int parts = L.ntiles <= 64 ? 8 : 1;
    const int64_t nb = (int64_t)L.nphase * L.nt * L.nt * (L.nt / z2) * parts;
    hipLaunchKernelGGL((k_fold_tiles<T>), dim3((unsigned)nb), dim3(256 * z2 / parts), 0, s, fa, norms, delta, noise);
  }
  kt_end(CNPC_KT_FOLD, s);
  CNPC_HIP(hipGetLastError());
  return CNPC_OK;
}

// sums and tile counts along with the sort (meshes of one bucket always)
static bool fused_sort(const PaintLayout& L) {
  return L.nbuckets == 1 || tune_value(CNPC_TUNE_SORT_FUSED) != 1;
}

cnpc_status launch_paint(const cnpc_mesh_desc* d, const uint32_t* gpos, const float* gw,
                         int64_t ngal, const uint32_t* rpos, const float* rw, int64_t nran,
                         const double* norms, void* delta, void* noise, void* ws, size_t ws_bytes,
                         hipStream_t s) {
  const bool weighted = (gw != nullptr) || (rw != nullptr);
  PaintLayout L = paint_layout(d, ngal, nran, weighted);
  if (ws_bytes < L.total) {
    set_error("paint workspace too small: need %zu bytes, got %zu", L.total, ws_bytes);
    return CNPC_EWORKSPACE;
  }
  unsigned char* w = reinterpret_cast<unsigned char*>(ws);
  // one bucket: paint_small; several: the bucket pass (one read of the catalog for the
  // tile counts and the first sort step) or, by the knob, the tile count in a read of
  // its own (the l = 0 sums of the first two are not used here)
  const int lm = fused_sort(L) ? 0 : -1;
  double* sums = reinterpret_cast<double*>(w + L.off_sums);
  if (d->dtype == CNPC_F64)
    return paint_t<double>(d, gpos, gw, ngal, rpos, rw, nran, norms, (double*)delta, (double*)noise, w,
                           L, false, s, lm, sums, sums + CNPC_SUMS_LEN, true, false);
  return paint_t<float>(d, gpos, gw, ngal, rpos, rw, nran, norms, (float*)delta, (float*)noise, w, L,
                        false, s, lm, sums, sums + CNPC_SUMS_LEN, true, false);
}

bool has_fold_zr2c(const cnpc_mesh_desc* d) {
  return d->interlace && d->n == 256 && fft_register_passes();
}

template <typename T>
static cnpc_status fold_zr2c_t(const cnpc_mesh_desc* d, const PaintLayout& L, unsigned char* ws,
                               const double* norms, cx<T>* dsp, cx<T>* nw1, int m, hipStream_t s) {
  FoldArgs<T> fa;
  fa.n = d->n;
  fa.nt = L.nt;
  fa.nphase = L.nphase;
  fa.nsets = L.nsets;
  for (int k = 0; k < L.nsets; ++k) fa.blocks[k] = reinterpret_cast<T*>(ws + L.off_blocks[k]);
  // one workgroup per (phase, tile column, x node of the tile)
  const int64_t grid = (int64_t)L.nphase * L.nt * L.nt * TILE;
  const size_t lds = sizeof(cx<T>) * (256 + (size_t)16 * FZ_RS);
  CNPC_TRY(ensure_twiddles());
  kt_begin(CNPC_KT_FOLD, s);
  hipLaunchKernelGGL((k_fold_zr2c<T>), dim3((unsigned)grid), dim3(256), lds, s, fa, norms, dsp, d->n / 2, nw1, m);
  kt_end(CNPC_KT_FOLD, s);
  CNPC_HIP(hipGetLastError());
  return CNPC_OK;
}

cnpc_status launch_paint_blocks_zr2c(const cnpc_mesh_desc* d, const uint32_t* gpos, const float* gw, int64_t ngal,
                                     const uint32_t* rpos, const float* rw, int64_t nran, int sums_lmax,
                                     double* gsums, double* rsums, double* norms, void* dsp, void* nw1, int m,
                                     void* ws, size_t ws_bytes, hipStream_t s) {
  const bool weighted = (gw != nullptr) || (rw != nullptr);
  PaintLayout L = paint_layout(d, ngal, nran, weighted);
  if (ws_bytes < L.total) {
    set_error("paint workspace too small: need %zu bytes, got %zu", L.total, ws_bytes);
    return CNPC_EWORKSPACE;
  }
  if (!has_fold_zr2c(d)) {
    set_error("fused fold and z pass: unsupported mesh");
    return CNPC_EUNSUPPORTED;
  }
  unsigned char* w = reinterpret_cast<unsigned char*>(ws);
  const bool fused = fused_sort(L);
  if (!fused) {
    // sums and tile counts in a pass of their own, norms before the painting
    uint32_t* count0 = reinterpret_cast<uint32_t*>(w + L.off_count[0]);
    uint32_t* count1 = reinterpret_cast<uint32_t*>(w + L.off_count[1]);
    double* partial = reinterpret_cast<double*>(w + L.off_partial);
    hipLaunchKernelGGL(k_zero_u32, dim3(64), dim3(256), 0, s, count0, (int64_t)L.ntiles);
    hipLaunchKernelGGL(k_zero_u32, dim3(64), dim3(256), 0, s, count1, (int64_t)L.ntiles);
    CNPC_HIP(hipGetLastError());
    CountArgs ca;
    ca.g = tile_geom(d);
    ca.ntiles = L.ntiles;
    ca.count = count0;
    CNPC_TRY(sums_counted(d, gpos, gw, ngal, sums_lmax, gsums, partial, ca, s));
    ca.count = count1;
    CNPC_TRY(sums_counted(d, rpos, rw, nran, sums_lmax, rsums, partial, ca, s));
    CNPC_TRY(launch_norms(d, gsums, rsums, ngal, norms, s));
  }
  const int lm = fused ? sums_lmax : -1;
  if (d->dtype == CNPC_F64) {
    CNPC_TRY(paint_t<double>(d, gpos, gw, ngal, rpos, rw, nran, norms, nullptr, nullptr, w, L, !fused, s, lm,
                             gsums, rsums, false));
    return fold_zr2c_t<double>(d, L, w, norms, (cx<double>*)dsp, (cx<double>*)nw1, m, s);
  }
  CNPC_TRY(paint_t<float>(d, gpos, gw, ngal, rpos, rw, nran, norms, nullptr, nullptr, w, L, !fused, s, lm, gsums,
                          rsums, false));
  return fold_zr2c_t<float>(d, L, w, norms, (cx<float>*)dsp, (cx<float>*)nw1, m, s);
}

cnpc_status launch_paint_fkp(const cnpc_mesh_desc* d, const uint32_t* gpos, const float* gw,
                             int64_t ngal, const uint32_t* rpos, const float* rw, int64_t nran,
                             int sums_lmax, double* gsums, double* rsums, double* norms, void* delta,
                             void* noise, void* ws, size_t ws_bytes, hipStream_t s) {
  const bool weighted = (gw != nullptr) || (rw != nullptr);
  PaintLayout L = paint_layout(d, ngal, nran, weighted);
  if (ws_bytes < L.total) {
    set_error("paint workspace too small: need %zu bytes, got %zu", L.total, ws_bytes);
    return CNPC_EWORKSPACE;
  }
  unsigned char* w = reinterpret_cast<unsigned char*>(ws);
  double* gs_ = gsums ? gsums : reinterpret_cast<double*>(w + L.off_sums);
  double* rs_ = rsums ? rsums : reinterpret_cast<double*>(w + L.off_sums) + CNPC_SUMS_LEN;
  if (fused_sort(L)) {
    if (d->dtype == CNPC_F64)
      return paint_t<double>(d, gpos, gw, ngal, rpos, rw, nran, norms, (double*)delta, (double*)noise, w, L,
                             false, s, sums_lmax, gs_, rs_);
    return paint_t<float>(d, gpos, gw, ngal, rpos, rw, nran, norms, (float*)delta, (float*)noise, w, L, false,
                          s, sums_lmax, gs_, rs_);
  }
  uint32_t* count0 = reinterpret_cast<uint32_t*>(w + L.off_count[0]);
  uint32_t* count1 = reinterpret_cast<uint32_t*>(w + L.off_count[1]);
  double* partial = reinterpret_cast<double*>(w + L.off_partial);
  double* gs = gsums ? gsums : reinterpret_cast<double*>(w + L.off_sums);
  double* rs = rsums ? rsums : reinterpret_cast<double*>(w + L.off_sums) + CNPC_SUMS_LEN;
  hipLaunchKernelGGL(k_zero_u32, dim3(64), dim3(256), 0, s, count0, (int64_t)L.ntiles);
  hipLaunchKernelGGL(k_zero_u32, dim3(64), dim3(256), 0, s, count1, (int64_t)L.ntiles);
  CNPC_HIP(hipGetLastError());
  CountArgs ca;
  ca.g = tile_geom(d);
  ca.ntiles = L.ntiles;
  ca.count = count0;
  CNPC_TRY(sums_counted(d, gpos, gw, ngal, sums_lmax, gs, partial, ca, s));
  ca.count = count1;
  CNPC_TRY(sums_counted(d, rpos, rw, nran, sums_lmax, rs, partial, ca, s));
  CNPC_TRY(launch_norms(d, gs, rs, ngal, norms, s));
  if (d->dtype == CNPC_F64)
    return paint_t<double>(d, gpos, gw, ngal, rpos, rw, nran, norms, (double*)delta, (double*)noise, w,
                           L, true, s);
  return paint_t<float>(d, gpos, gw, ngal, rpos, rw, nran, norms, (float*)delta, (float*)noise, w, L,
                        true, s);
}

}  // namespace cnpc
