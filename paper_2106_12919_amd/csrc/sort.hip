// Counting sort of particles by grid tile (support for the tiled deposition).
//
// Tiles are kTile^3 blocks of cells (partial at the upper end of an axis); particles
// with an out-of-range cell index go to one extra bucket after the last tile so
// the sorted order has no holes (they are counted and never deposited).  Three
// launches: count per tile, exclusive scan of the counts, rank (each particle's
// slot in tile order, kept as the permutation slot -> particle).
#include <algorithm>

#include "kernels.h"

namespace pic {

namespace {

__device__ inline uint32_t fdiv(uint32_t n, const FastDiv& f) { return (__umulhi(n, f.m) + n) >> f.s; }

__device__ inline int tile_key(int c, const GridGeom& g, const TileGeom& t) {
  if (c < 0 || c >= g.nx * g.ny * g.nz) return t.ntiles;
  const int r = (int)fdiv((uint32_t)c, g.nz_div);
  const int k = c - r * g.nz;
  const int i = (int)fdiv((uint32_t)r, g.ny_div);
  const int j = r - i * g.ny;
  return ((i / kTile) * t.nty + j / kTile) * t.ntz + k / kTile;
}

// A workgroup counts its BLOCK * kSortPer particles per tile in an LDS table and touches each global
// counter once per tile it holds.  Up to kSortBuckets buckets (128 KiB of LDS) the table is indexed by
// the tile; beyond, by a hash with linear probing (HASH): particles are nearly grouped by tile (the
// previous call's order), so a workgroup holds few distinct tiles.  A key that finds no place in the
// table goes to the global counter by itself.  32769 buckets, 134 M particles (256^3, 8 per cell) in cell order:
// count and rank 368 + 523 us, against 512 + 656 (and 318 to invert the slots) with one global atomic per wave
// and tile; moved by up to 8 cells 793 + 1042, against 1926 + 2228 (and 481).
// At 1025 and 6157 buckets the hash was slower than the indexed table (33 against 26 us for 2.1 M grouped
// particles, 407 against 341 for 9 M scattered ones).
constexpr int kSortPer = 8;
constexpr int kSortBuckets = 32768;
constexpr int kSortTable = 2048;  // entries of the hashed table
constexpr int kSortProbes = 16;

template <bool HASH>
__device__ inline int table_place(volatile int* keys, int key) {
  if (!HASH) return key;
  const unsigned h = ((unsigned)key * 2654435761u) >> 21;  // 11 bits: kSortTable entries
#pragma unroll 1
  for (int p = 0; p < kSortProbes; ++p) {
    const int e = (int)((h + p) & (kSortTable - 1));
    int k = keys[e];
    if (k < 0) k = atomicCAS(const_cast<int*>(keys) + e, -1, key);
    if (k < 0 || k == key) return e;
  }
  return -1;
}

// Adds one per valid lane to the table entry of its key (global[key] when the table has no place):
// place = the entry or -1, returns the lane's rank in it (the global slot when place < 0; ranks only
// when RANK).  The first few distinct keys of a wave are added by one lane each for all lanes of the
// key (grouped particles: one or two keys per wave); lanes left after that (scattered particles) add
// for themselves.
template <bool HASH, bool RANK>
__device__ inline int table_add(int* keys, int* cnt, int* global, int key, bool valid, int& place) {
  constexpr int kGrouped = 3;
  unsigned long long active = __ballot(valid);
  const int lane = __lane_id();
  int leader_of = lane, rank = 0, group = valid ? 1 : 0;
  for (int q = 0; q < kGrouped && active; ++q) {
    const int leader = __ffsll((unsigned long long)active) - 1;
    const int lkey = __shfl(key, leader);
    const unsigned long long same = __ballot(valid && key == lkey) & active;
    if ((same >> lane) & 1ull) {
      leader_of = leader;
      rank = __popcll(same & ((1ull << lane) - 1ull));
      group = lane == leader ? __popcll(same) : 0;
    }
    active &= ~same;
  }
  int base = 0;
  place = -1;
  if (group > 0) {
    place = table_place<HASH>(keys, key);
    base = atomicAdd(place >= 0 ? &cnt[place] : &global[key], group);
  }
  if (!RANK) return 0;
  base = __shfl(base, leader_of);
  place = __shfl(place, leader_of);
  return base + rank;
}

template <bool HASH, int BLOCK>
__device__ inline void table_clear(int* keys, int* cnt, int nbk) {
  for (int e = threadIdx.x; e < (HASH ? kSortTable : nbk); e += BLOCK) {
    cnt[e] = 0;
    if (HASH) keys[e] = -1;
  }
  __syncthreads();
}

// Dynamic LDS of both: the counts (the table's entries, or one per bucket), then with HASH the keys and one
// more int.
template <bool HASH, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_tile_count(GridGeom g, TileGeom t, const int32_t* __restrict__ cell,
                                                           long long n, int* counts) {
  extern __shared__ int cnt[];
  int* const keys = cnt + kSortTable;
  const int nbk = t.ntiles + 1;
  table_clear<HASH, BLOCK>(keys, cnt, nbk);
  const long long p0 = (long long)blockIdx.x * BLOCK * kSortPer + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const long long p = p0 + (long long)u * BLOCK;
    const int key = (p < n) ? tile_key(cell[p], g, t) : 0;
    int place;
    (void)table_add<HASH, false>(keys, cnt, counts, key, p < n, place);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < (HASH ? kSortTable : nbk); e += BLOCK) {
    const int c = cnt[e];
    if (c) atomicAdd(&counts[HASH ? keys[e] : e], c);
  }
}

// Each workgroup reserves one run per tile on ``cursor`` and places its particles in it by rank.  With ``slots``
// (HASH), a workgroup that fills seven eighths of its table (an unordered species)
// writes the slots of its particles in order and says so in scattered[block], for k_tile_place: in one kernel
// with that many global atomics the scattered writes of perm are slow (134 M unordered particles in 32769
// buckets: count, rank and place 12.5 ms, with one rank kernel 17.6).
template <bool HASH, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_tile_rank(GridGeom g, TileGeom t, const int32_t* __restrict__ cell,
                                                          long long n, int* cursor, int* perm, int* bad, int* slots,
                                                          int* scattered) {
  extern __shared__ int cnt[];
  int* const keys = cnt + kSortTable;
  int* const used = keys + kSortTable;  // (HASH) entries of the table in use
  const int nbk = t.ntiles + 1;
  if (HASH && threadIdx.x == 0) *used = 0;
  table_clear<HASH, BLOCK>(keys, cnt, nbk);
  const long long p0 = (long long)blockIdx.x * BLOCK * kSortPer + threadIdx.x;
  int place[kSortPer], rank[kSortPer];
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const long long p = p0 + (long long)u * BLOCK;
    const int key = (p < n) ? tile_key(cell[p], g, t) : 0;
    rank[u] = table_add<HASH, true>(keys, cnt, cursor, key, p < n, place[u]);
    if (p < n && key == t.ntiles && bad) atomicAdd(bad, 1);
  }
  __syncthreads();
  if (HASH) {
    int mine = 0;
#pragma unroll
    for (int e = threadIdx.x; e < kSortTable; e += BLOCK) mine += __popcll(__ballot(cnt[e] != 0));
    if (mine && __lane_id() == 0) atomicAdd(used, mine);
  }
  for (int e = threadIdx.x; e < (HASH ? kSortTable : nbk); e += BLOCK) {
    const int c = cnt[e];
    if (c) cnt[e] = atomicAdd(&cursor[HASH ? keys[e] : e], c);  // this workgroup's run of the tile
  }
  __syncthreads();
  const bool split = HASH && slots && __builtin_amdgcn_readfirstlane(*used) > kSortTable / 8 * 7;
  if (HASH && slots && threadIdx.x == 0) scattered[blockIdx.x] = split;
  int* const out = split ? slots : perm;
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const long long p = p0 + (long long)u * BLOCK;
    const int slot = (place[u] >= 0 ? cnt[place[u]] : 0) + rank[u];
    if (p < n) out[split ? (int)p : slot] = split ? slot : (int)p;
  }
}

// The particles of the workgroups that k_tile_rank found scattered, to their slots.  The resident workgroups
// walk the particles side by side, BLOCK at a time (64 flags a look), so that what they write at one time
// is a short run in each tile.
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_tile_place(long long n, const int* __restrict__ slots,
                                                      const int* __restrict__ scattered, int* perm) {
  const long long chunks = (n + BLOCK - 1) / BLOCK, step = gridDim.x;
  for (long long c0 = blockIdx.x; c0 < chunks; c0 += 64 * step) {
    const long long c = c0 + __lane_id() * step;
    unsigned long long todo = __ballot(c < chunks && scattered[c / kSortPer] != 0);
    for (; todo; todo &= todo - 1) {
      const long long p = (c0 + (__ffsll(todo) - 1) * step) * BLOCK + threadIdx.x;
      if (p < n) perm[slots[p]] = (int)p;
    }
  }
}

// Exclusive scan of counts[0..m) into starts[0..m] (starts[m] = the total) and cursor[0..m)
// by blocks of 1024 threads, in chunks of 1024 x PER entries: thread t takes the PER adjacent
// entries at the chunk's base + PER t as 16-byte vectors, and the block scans the thread sums (a scan
// within each wave, then over the 16 wave totals).  A scan leaves the counts at zero, for the next
// count into them.
constexpr int kScanPer = 8;
constexpr int kScanChunk = 1024 * kScanPer;
constexpr int kScanWaves = 1024 / 64;

// One chunk from ``carry`` (the sum of everything before it); returns the sum up to its end.
// Every thread of the block calls it.
template <int PER>
__device__ inline int scan_chunk(int* counts, int* starts, int* cursor, int m, int base, int carry, int* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = base + tid * PER;
  int v[PER];
  const bool whole = i0 + PER <= m;
  if (whole) {
#pragma unroll
    for (int k = 0; k < PER; k += 4) {
      const int4 q = *reinterpret_cast<const int4*>(counts + i0 + k);
      v[k] = q.x; v[k + 1] = q.y; v[k + 2] = q.z; v[k + 3] = q.w;
      *reinterpret_cast<int4*>(counts + i0 + k) = make_int4(0, 0, 0, 0);
    }
  } else {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      v[k] = (i0 + k < m) ? counts[i0 + k] : 0;
      if (i0 + k < m) counts[i0 + k] = 0;
    }
  }
  int s = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) s += v[k];
  int x = s;  // inclusive scan of the thread sums within the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  int run = carry + x - s, total = carry;
#pragma unroll
  for (int w = 0; w < kScanWaves; ++w) {
    run += w < wave ? wsum[w] : 0;
    total += wsum[w];
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int c = v[k];
    v[k] = run;
    run += c;
  }
  if (whole) {
#pragma unroll
    for (int k = 0; k < PER; k += 4) {
      const int4 q = make_int4(v[k], v[k + 1], v[k + 2], v[k + 3]);
      *reinterpret_cast<int4*>(starts + i0 + k) = q;
      *reinterpret_cast<int4*>(cursor + i0 + k) = q;
    }
  } else {
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (i0 + k < m) {
        starts[i0 + k] = v[k];
        cursor[i0 + k] = v[k];
      }
  }
  return total;
}

// m <= 1024 x PER, one block (one launch beats three there).
template <int PER>
__global__ void __launch_bounds__(1024) k_scan(int* counts, int* starts, int* cursor, int m) {
  __shared__ int wsum[kScanWaves];
  const int total = scan_chunk<PER>(counts, starts, cursor, m, 0, 0, wsum);
  if (threadIdx.x == 0) starts[m] = total;
}

// Large m, first of three launches: sums[b] = the total of chunk b.
__global__ void __launch_bounds__(1024) k_scan_sums(const int* __restrict__ counts, int m, int* sums) {
  __shared__ int wsum[kScanWaves];
  const int base = blockIdx.x * kScanChunk, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int s = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    const int i = base + k * 1024 + (int)threadIdx.x;
    if (i < m) s += counts[i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) wsum[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < kScanWaves; ++w) t += wsum[w];
    sums[blockIdx.x] = t;
  }
}

// Second launch (one block, nb <= 1024): sums -> their exclusive scan in place; *total = the sum.
__global__ void __launch_bounds__(1024) k_scan_offsets(int* sums, int nb, int* total) {
  __shared__ int wsum[kScanWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int v = tid < nb ? sums[tid] : 0;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  if (tid < nb) sums[tid] = before + x - v;
  if (tid == 1023) *total = before + x;
}

// Third launch: block b scans chunk b from its offset.
__global__ void __launch_bounds__(1024) k_scan_apply(int* counts, int* starts, int* cursor, int m,
                                                     const int* __restrict__ offsets) {
  __shared__ int wsum[kScanWaves];
  (void)scan_chunk<kScanPer>(counts, starts, cursor, m, blockIdx.x * kScanChunk, offsets[blockIdx.x], wsum);
}

// For every destination tile D of the new grouping: the slot runs of the particles that
// arrive from each neighbour source tile S (grouped by S in the previous step), in the
// order of the 27 offsets, from starts[D]; bases[27 S + nb] receives the start of the run
// of S's particles whose offset to D is nb, cursor[D] the first slot after all runs.
// An offset that names the same S as another (grids of one or two tiles along an axis)
// is taken once, with the index the particle kernels compute for it.
// One 32-lane group per destination tile D; lane o < 27 takes the offset o, its source
// tile and count, and a scan across the group places the runs.
__global__ void __launch_bounds__(256) k_neighbour_bases(TileGeom t, const int* __restrict__ old_starts,
                                                         const int* __restrict__ nbr_counts,
                                                         const int* __restrict__ new_starts, int* bases, int* cursor) {
  const int D = (blockIdx.x * blockDim.x + threadIdx.x) >> 5;
  const int o = threadIdx.x & 31;
  if (D >= t.ntiles) return;  // whole 32-lane groups leave together
  const int dz = D % t.ntz, dy = (D / t.ntz) % t.nty, dx = D / (t.ntz * t.nty);
  const int nt[3] = {t.ntx, t.nty, t.ntz};
  const int dc[3] = {dx, dy, dz};
  const int off[3] = {o / 9 - 1, (o / 3) % 3 - 1, o % 3 - 1};
  int sc[3], canon = 0;
  for (int a = 0; a < 3; ++a) {
    sc[a] = (dc[a] - off[a] + nt[a]) % nt[a];
    int d = dc[a] - sc[a];  // as the particle kernels wrap it
    if (d > 1) d -= nt[a];
    if (d < -1) d += nt[a];
    canon = canon * 3 + (d + 1);
  }
  const int S = (sc[0] * t.nty + sc[1]) * t.ntz + sc[2];
  const bool take = o < 27 && canon == o;
  const int Sv = take ? S : 0;
  const int s0 = old_starts[Sv], s1 = old_starts[Sv + 1];  // an empty tile published no counts
  const int cv = nbr_counts[27 * Sv + (take ? o : 0)];
  const int c = (take && s0 != s1) ? cv : 0;
  int x = c;  // inclusive scan over the group
  for (int k = 1; k < 32; k <<= 1) {
    const int y = __shfl_up(x, k, 32);
    if (o >= k) x += y;
  }
  const int run0 = new_starts[D];
  if (take && s0 != s1) bases[27 * S + o] = run0 + x - c;
  if (o == 31) cursor[D] = run0 + x;
}

}  // namespace

FastDiv make_fastdiv(uint32_t d) {
  FastDiv f{d, 0u, 0u};
  while ((1ull << f.s) < d) ++f.s;
  f.m = (uint32_t)((((1ull << 32) * ((1ull << f.s) - d)) / d) + 1);
  return f;
}

GridGeom make_geom(int nx, int ny, int nz, double dx, double dy, double dz, double dt, int shape_order) {
  GridGeom g{nx, ny, nz, dx, dy, dz, dt, shape_order, make_fastdiv((uint32_t)ny), make_fastdiv((uint32_t)nz),
             0.0, 0.0, 0.0, 0};
  return g;
}

TileGeom make_tiles(const GridGeom& g) {
  TileGeom t{};
  t.ntx = (g.nx + kTile - 1) / kTile;
  t.nty = (g.ny + kTile - 1) / kTile;
  t.ntz = (g.nz + kTile - 1) / kTile;
  t.ntiles = t.ntx * t.nty * t.ntz;
  t.distinct = g.nx % kTile == 0 && g.ny % kTile == 0 && g.nz % kTile == 0 && t.ntx > 2 && t.nty > 2 && t.ntz > 2;
  return t;
}

// The exclusive scan of the ntiles + 1 bucket counts: one block up to 16384 entries, else
// the three-launch form through t.scan_tmp (at most 257 chunks on a 1024^3 grid).
void scan_counts(const TileGeom& t, int* counts, int* starts, int* cursor, hipStream_t s) {
  const int m = t.ntiles + 1;
  const int nb = (m + kScanChunk - 1) / kScanChunk;
  if (nb <= 2) {
    if (m <= 4096) hipLaunchKernelGGL(k_scan<4>, dim3(1), dim3(1024), 0, s, counts, starts, cursor, m);
    else hipLaunchKernelGGL(k_scan<16>, dim3(1), dim3(1024), 0, s, counts, starts, cursor, m);
    return;
  }
  hipLaunchKernelGGL(k_scan_sums, dim3(nb), dim3(1024), 0, s, (const int*)counts, m, t.scan_tmp);
  hipLaunchKernelGGL(k_scan_offsets, dim3(1), dim3(1024), 0, s, t.scan_tmp, nb, starts + m);
  hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(1024), 0, s, counts, starts, cursor, m, (const int*)t.scan_tmp);
}

namespace {

template <bool HASH, int BLOCK>
void sort_with(const GridGeom& g, const TileGeom& t, const int32_t* cell, int64_t n, int* counts, int* starts,
               int* cursor, int* perm, int* bad, hipStream_t s) {
  const dim3 grid((unsigned)((n + BLOCK * kSortPer - 1) / (BLOCK * kSortPer))), block(BLOCK);
  const size_t lds = sizeof(int) * (size_t)(HASH ? 2 * kSortTable + 1 : t.ntiles + 1);
  allow_lds((const void*)k_tile_count<HASH, BLOCK>, lds);
  allow_lds((const void*)k_tile_rank<HASH, BLOCK>, lds);
  if (n > 0)
    hipLaunchKernelGGL((k_tile_count<HASH, BLOCK>), grid, block, lds, s, g, t, cell, (long long)n, counts);
  scan_counts(t, counts, starts, cursor, s);
  if (n <= 0) return;
  int* const slots = HASH && t.spare && (size_t)n + grid.x <= t.spare_ints ? t.spare : nullptr;
  int* const scattered = slots ? slots + n : nullptr;
  hipLaunchKernelGGL((k_tile_rank<HASH, BLOCK>), grid, block, lds, s, g, t, cell, (long long)n, cursor, perm, bad, slots,
                     scattered);
  if (slots)
    hipLaunchKernelGGL(k_tile_place<BLOCK>, dim3(std::min(grid.x * kSortPer, 1024u)), block, 0, s, (long long)n,
                       (const int*)slots, (const int*)scattered, perm);  // 4 workgroups per CU
}

}  // namespace

void tile_sort(const GridGeom& g, const TileGeom& t, const int32_t* cell, int64_t n, int* counts, int* starts,
               int* cursor, int* perm, int* bad, hipStream_t s) {
  // buckets 0..ntiles-1 are tiles, bucket ntiles collects invalid cells; small tables (and the hashed
  // one) take small workgroups, large ones as many particles per table as a workgroup can hold
  if (t.ntiles + 1 > kSortBuckets) sort_with<true, 512>(g, t, cell, n, counts, starts, cursor, perm, bad, s);
  else if (t.ntiles + 1 > 1024) sort_with<false, 1024>(g, t, cell, n, counts, starts, cursor, perm, bad, s);
  else sort_with<false, 256>(g, t, cell, n, counts, starts, cursor, perm, bad, s);
}

void neighbour_bases(const TileGeom& t, const int* old_starts, const int* nbr_counts, const int* new_starts,
                     int* bases, int* cursor, hipStream_t s) {
  hipLaunchKernelGGL(k_neighbour_bases, dim3((unsigned)((t.ntiles + 7) / 8)), dim3(256), 0, s, t, old_starts,
                     nbr_counts, new_starts, bases, cursor);
}

}  // namespace pic
