// Closed counts of all edges from the triangles of the graph, and the
// clustering steps that follow from exact counts.
//
// With the vertices ordered by degree and every edge (u, v) kept in the row of
// its lower-degree endpoint u, a triangle is one u with two entries v, w of
// its row that are adjacent, so the pairs of entries of all rows are the only
// candidates: sum of D(D-1)/2 over rows of length D, where the intersections
// of kernels.hip read sum of min(d(u), d(v)) elements (R-MAT scale 22: 7.2 G
// against 43 G for exact counts, and 28.9 / 11.1 / 3.3 G with every early
// exit at eps = 1/5, 1/2, 4/5).
//
// A triangle u, v, w (in order of the columns of u and v) counts for three
// edges, and none of the three needs an atomic per triangle on global memory:
//   (v, w)  count kernels: row v is held in LDS with a counter per entry; the
//           columns of every in-edge (u, v) after v's own are looked up in it,
//           a hit adds to the entry's counter, and the counters of a job are
//           added to row v of cnt once;
//   (u, v), (u, w)  the same lookups, as one bit per column, are written to
//           row u's triangle of bits (0.9 GB for the 7.2 G pairs).  The close
//           kernel adds, for every entry of row u, the bits of its row and of
//           its column.
#include "tri.h"
#include "device.h"

#include <algorithm>
#include <climits>
#include <type_traits>
#include <utility>
#include <vector>

namespace scan {
namespace {

__host__ __device__ inline uint32_t tri_lines(int32_t D) { return (uint32_t)(D + kTriLine - 1) / kTriLine; }

// Words of row u's bits before those of column i (rows of W lines: column i
// keeps the words of lines i / 32 .. W - 1).
__host__ __device__ inline uint32_t tri_word(uint32_t W, uint32_t i) {
  const uint32_t b = i >> 5;
  return i * W - (32 * (b * (b - 1) / 2) + (i & 31) * b);
}

// ---------------------------------------------------------------------------
// Layout

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane == 0 ? 0ull : (~0ull >> (64 - lane)); }

// Rows above kTriBigRow arcs are taken by a block per kTriBigChunk of them, which
// add up or append through the row's counters (one block per row walked the
// longest one, 163,089 arcs on R-MAT scale 22, 160 dependent rounds long); the
// others by a wave.
struct BigChunk {
  int32_t h, id;
  int64_t begin, end;  // arcs
};
constexpr int64_t kTriBigRow = kLongRow;
constexpr int64_t kTriBigChunk = 2048;

__global__ __launch_bounds__(256) void k_row_len_block(const BigChunk* chunks, const int32_t* ci, const int32_t* hof,
                                                       int32_t* row) {
  __shared__ int32_t sum;
  const BigChunk C = chunks[blockIdx.x];
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  int32_t c = 0;
  for (int64_t k = C.begin + threadIdx.x; k < C.end; k += 256) c += hof[ci[k]] < C.h ? 1 : 0;
  c = (int32_t)wave_sum((unsigned long long)c);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(&sum, c);
  __syncthreads();
  if (threadIdx.x == 0 && sum) atomicAdd(row + C.h, sum);
}

// Renaming: a stable sort of the vertices by max degree - degree, 8 bits a pass
// (one pass up to degree 255, three for any R-MAT), a block per kSortTile
// consecutive ones.  (On one host thread, faulting the arrays in and two passes
// over the vertices took most of the creation of a large sparse graph: a road-like
// grid of 4 million vertices 22.5 ms, now 11.9; R-MAT scale 22 55 and 43.  Host
// threads came to 17.4 and 45, and made a process's first creation 3 ms longer.)
constexpr int kSortTile = 4096;
inline int64_t sort_blocks(int32_t n) { return ((int64_t)n + kSortTile - 1) / kSortTile; }
inline int64_t sort_counts(int32_t n) { return 256 * sort_blocks(n); }

// Vertex i of the pass: of the input, or of the graph.
__device__ __forceinline__ int2 sort_item(int64_t i, const int2* in, const int64_t* rp, int32_t max_degree) {
  return in ? in[i] : make_int2(max_degree - (int32_t)(rp[i + 1] - rp[i]), (int32_t)i);
}

// cnt[256 digits][blocks]
__global__ __launch_bounds__(256) void k_sort_count(int32_t n, int shift, const int64_t* rp, int32_t max_degree,
                                                    const int2* in, int64_t* cnt) {
  __shared__ uint32_t c[256];
  c[threadIdx.x] = 0;
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * kSortTile, e = min(b + kSortTile, (int64_t)n);
  for (int64_t i = b + threadIdx.x; i < e; i += 256) atomicAdd(&c[sort_item(i, in, rp, max_degree).x >> shift & 255], 1u);
  __syncthreads();
  cnt[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = c[threadIdx.x];
}

// Lanes of the wave whose valid digit is this lane's.
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid) {
  uint64_t m = __ballot(valid);
  for (int b = 0; b < 8; ++b) {
    const bool on = (d >> b) & 1u;
    const uint64_t v = __ballot(on);
    m &= on ? v : ~v;
  }
  return m;
}

// A wave places a quarter of the tile, 64 vertices at a time, behind the waves
// before it (off: the scanned counts); the last pass (out null) writes the names.
__global__ __launch_bounds__(256) void k_sort_place(int32_t n, int shift, const int64_t* rp, int32_t max_degree,
                                                    const int2* in, const int64_t* off, int2* out, int32_t* hof,
                                                    int32_t* idof) {
  __shared__ uint32_t at[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int w = 0; w < 4; ++w) at[w][threadIdx.x] = 0;
  __syncthreads();
  const int64_t b = (int64_t)blockIdx.x * kSortTile + wave * (kSortTile / 4);
  for (int r = 0; r < kSortTile / 256; ++r) {
    const int64_t i = b + r * 64 + lane;
    const bool valid = i < n;
    const uint32_t d = valid ? (uint32_t)(sort_item(i, in, rp, max_degree).x >> shift) & 255u : 0;
    const uint64_t m = same_digit(d, valid);
    if (valid && (m & lanes_below(lane)) == 0) at[wave][d] += (uint32_t)__popcll(m);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  {
    uint32_t to = (uint32_t)off[(int64_t)threadIdx.x * gridDim.x + blockIdx.x];
    for (int w = 0; w < 4; ++w) {
      const uint32_t c = at[w][threadIdx.x];
      at[w][threadIdx.x] = to;
      to += c;
    }
  }
  __syncthreads();
  for (int r = 0; r < kSortTile / 256; ++r) {
    const int64_t i = b + r * 64 + lane;
    const bool valid = i < n;
    const int2 x = valid ? sort_item(i, in, rp, max_degree) : make_int2(0, 0);
    const uint32_t d = (uint32_t)(x.x >> shift) & 255u;
    const uint64_t m = same_digit(d, valid);
    const uint32_t to = at[wave][d] + (uint32_t)__popcll(m & lanes_below(lane));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && (m & lanes_below(lane)) == 0) at[wave][d] += (uint32_t)__popcll(m);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (!valid) continue;
    if (out) {
      out[to] = x;
    } else {
      hof[x.y] = (int32_t)to;
      idof[to] = x.y;
    }
  }
}

// a, b: n items each; digits: 2 sort_counts(n); work: of their scan.
hipError_t sort_by_degree(hipStream_t s, int32_t n, const int64_t* rp, int32_t max_degree, int2* a, int2* b,
                          int64_t* digits, int64_t* work, int32_t* hof, int32_t* idof) {
  const unsigned grid = (unsigned)sort_blocks(n);
  int64_t* off = digits + sort_counts(n);
  const int2* in = nullptr;
  for (int shift = 0; shift == 0 || max_degree >> shift > 0; shift += 8) {
    const bool last = max_degree >> shift < 256;
    k_sort_count<<<grid, 256, 0, s>>>(n, shift, rp, max_degree, in, digits);
    const hipError_t e = exclusive_scan(s, digits, off, sort_counts(n), work);
    if (e != hipSuccess) return e;
    int2* out = last ? nullptr : in == a ? b : a;
    k_sort_place<<<grid, 256, 0, s>>>(n, shift, rp, max_degree, in, off, out, hof, idof);
    if (last) break;
    in = out;
  }
  return hipGetLastError();
}

// The same inside every graph of a batch, on the host.
void rename_groups(const int64_t* rp, const TriGroups& G, int32_t* hof) {
  std::vector<int32_t> first;
  for (int32_t k = 0; k < G.count; ++k) {
    const int32_t v0 = (int32_t)G.h_vtx_off[k], v1 = (int32_t)G.h_vtx_off[k + 1];
    int64_t most = 0;
    for (int32_t v = v0; v < v1; ++v) most = std::max(most, rp[v + 1] - rp[v]);
    first.assign((size_t)most + 1, 0);
    for (int32_t v = v0; v < v1; ++v) ++first[(size_t)(rp[v + 1] - rp[v])];
    int32_t acc = v0;
    for (int64_t d = most; d >= 0; --d) acc += std::exchange(first[(size_t)d], acc);
    for (int32_t v = v0; v < v1; ++v) hof[v] = first[(size_t)(rp[v + 1] - rp[v])]++;
  }
}

__global__ void k_inverse(int32_t n, const int32_t* hof, int32_t* idof) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x < n) idof[hof[x]] = (int32_t)x;
}

// Degrees by h; the length of the rows above kTriBigRow starts at 0.
__global__ void k_degrees(int32_t n, const int64_t* rp, const int32_t* idof, int32_t* deg, int32_t* row) {
  const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= n) return;
  const int32_t x = idof[h];
  deg[h] = (int32_t)(rp[x + 1] - rp[x]);
  row[h] = 0;
}

// The kernels below take G lanes per vertex: 64, or 8 for the vertices of at most
// kNarrowRow neighbours, which follow the others, where there are kNarrowWorth of
// them (a wave each, with 61 lanes idle, made each of the five kernels take 2.4 to
// 5.8 ms on a triangulated grid of 9 million vertices, all of degree 6, and its
// creation 32 ms, now 16; of a road-like grid of 4 million 11.9 and 6.3).
constexpr int32_t kNarrowWorth = 1 << 16;

// Vertex and lane of a thread.
template <int G>
__device__ __forceinline__ int64_t group_vertex(int32_t h0) {
  return h0 + ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
}

template <int G, typename T>
__device__ __forceinline__ T group_sum(T x) {
  for (int d = G / 2; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
  return x;
}

// The group's part of a ballot.
template <int G>
__device__ __forceinline__ uint64_t group_ballot(bool p) {
  const uint64_t m = __ballot(p);
  if constexpr (G == 64) return m;
  return (m >> (threadIdx.x & 63 & ~(G - 1))) & ((1ull << (G & 63)) - 1);
}

template <int G>
__global__ __launch_bounds__(256) void k_row_len_wave(int32_t h0, int32_t n, const int64_t* rp, const int32_t* ci,
                                                      const int32_t* hof, const int32_t* idof, int32_t* row) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t h = group_vertex<G>(h0);
  if (h >= n) return;
  const int32_t x = idof[h];
  const int64_t b = rp[x], e = rp[x + 1];
  int32_t c = 0;
  for (int64_t k = b + lane; k < e; k += G) c += hof[ci[k]] < h ? 1 : 0;
  c = group_sum<G>(c);
  if (lane == 0) row[h] = c;
}

// Room for the records of every vertex, from its in-edges' rows (a record's
// column is not known yet), and whether the wave kernel takes it.
__device__ __forceinline__ void tri_room(int32_t D, unsigned long long lines, unsigned long long recs, int64_t* nin,
                                         uint8_t* wave) {
  const bool w = D <= kTriWaveRow && lines <= kTriWaveWords;
  *wave = w;
  *nin = (int64_t)(w ? lines : recs);
}

__global__ __launch_bounds__(256) void k_in_room_block(const BigChunk* chunks, const int32_t* ci, const int32_t* hof,
                                                       const int32_t* row, unsigned long long* room) {
  __shared__ unsigned long long sum, sumr;
  const BigChunk C = chunks[blockIdx.x];
  if (threadIdx.x == 0) sum = sumr = 0;
  __syncthreads();
  unsigned long long c = 0, r = 0;
  for (int64_t k = C.begin + threadIdx.x; k < C.end; k += 256) {
    const int32_t u = hof[ci[k]];
    const uint32_t W = u > C.h && row[u] > 1 ? tri_lines(row[u]) : 0;
    c += W;
    r += (W + kTriRecLines - 1) / kTriRecLines;
  }
  c = wave_sum(c);
  r = wave_sum(r);
  if ((threadIdx.x & 63) == 0 && c) {
    atomicAdd(&sum, c);
    atomicAdd(&sumr, r);
  }
  __syncthreads();
  if (threadIdx.x == 0 && sum) {
    atomicAdd(room + 2 * C.h, sum);
    atomicAdd(room + 2 * C.h + 1, sumr);
  }
}

// room[2 h], room[2 h + 1]: lines and records of the rows above kTriBigRow.
__global__ void k_in_room_big(int32_t nbig, const int32_t* row, const unsigned long long* room, int64_t* nin,
                              uint8_t* wcls) {
  const int32_t h = blockIdx.x * blockDim.x + threadIdx.x;
  if (h < nbig) tri_room(row[h], room[2 * h], room[2 * h + 1], nin + h, wcls + h);
}

template <int G>
__global__ __launch_bounds__(256) void k_in_room_wave(int32_t h0, int32_t n, const int64_t* rp, const int32_t* ci,
                                                      const int32_t* hof, const int32_t* idof, const int32_t* row,
                                                      int64_t* nin, uint8_t* wcls) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t h = group_vertex<G>(h0);
  if (h >= n) return;
  const int32_t x = idof[h];
  const int64_t b = rp[x], e = rp[x + 1];
  unsigned long long c = 0, r = 0;
  for (int64_t k = b + lane; k < e; k += G) {
    const int32_t u = hof[ci[k]];
    const uint32_t W = u > h && row[u] > 1 ? tri_lines(row[u]) : 0;
    c += W;
    r += (W + kTriRecLines - 1) / kTriRecLines;
  }
  c = group_sum<G>(c);
  r = group_sum<G>(r);
  if (lane == 0) tri_room(row[h], c, r, nin + h, wcls + h);
}

// Per vertex: lines and bit words of its row; all entries, and the longest row.
// (A grid-stride loop: one atomic per wave of 64 vertices queued on one address.)
__global__ void k_row_sizes(int32_t n, const int32_t* row, int64_t* nline, int64_t* nword, unsigned long long* entries,
                            int32_t* max_row) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  unsigned long long all = 0;
  int32_t m = 0;
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h <= n; h += stride) {
    const int32_t D = h < n ? row[h] : 0;
    const uint32_t W = tri_lines(D);
    nline[h] = W;
    nword[h] = D <= kTriMaxRow ? tri_word(W, (uint32_t)D) : 0;
    all += (unsigned long long)D;
    m = max(m, D);
  }
  all = wave_sum(all);
  for (int d = 32; d >= 1; d >>= 1) m = max(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) {
    if (all) atomicAdd(entries, all);
    if (m > 0) atomicMax(max_row, m);
  }
}

__global__ void k_narrow(int32_t n, const int64_t* a, const int64_t* b, uint32_t* x, uint32_t* y) {
  const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (h > n) return;
  x[h] = (uint32_t)a[h];
  y[h] = (uint32_t)b[h];
}

// Entries of every row (sorted afterwards); at[h] counts those of the rows above
// kTriBigRow.
__global__ __launch_bounds__(256) void k_row_fill_block(const BigChunk* chunks, const int32_t* ci, const int32_t* hof,
                                                        const uint32_t* oline, const int32_t* row, uint32_t* at,
                                                        int32_t* oc) {
  const BigChunk C = chunks[blockIdx.x];
  const int lane = threadIdx.x & 63;
  const int32_t D = row[C.h];
  int32_t* out = oc + (int64_t)oline[C.h] * kTriLine;
  for (int64_t k0 = C.begin; k0 < C.end; k0 += 256) {
    const int64_t k = k0 + threadIdx.x;
    const int32_t y = k < C.end ? hof[ci[k]] : INT_MAX;
    const bool keep = y < C.h;
    const uint64_t mask = __ballot(keep);
    uint32_t base = 0;
    if (lane == 0 && mask) base = atomicAdd(at + C.h, (uint32_t)__popcll(mask));
    base = __shfl(base, 0, 64);
    const int32_t p = (int32_t)(base + (uint32_t)__popcll(mask & lanes_below(lane)));
    if (keep && p < D) out[p] = y + 1;
  }
}

// Padding of the rows above kTriBigRow.
__global__ void k_row_pad(int32_t nbig, const uint32_t* oline, const int32_t* row, int32_t* oc) {
  const int32_t h = (blockIdx.x * blockDim.x + threadIdx.x) >> 5;
  if (h >= nbig) return;
  const int32_t D = row[h], p = D + (int32_t)(threadIdx.x & 31);
  if (p < (int32_t)tri_lines(D) * kTriLine) oc[(int64_t)oline[h] * kTriLine + p] = 0;
}

template <int G>
__global__ __launch_bounds__(256) void k_row_fill_wave(int32_t h0, int32_t n, const int64_t* rp, const int32_t* ci,
                                                       const int32_t* hof, const int32_t* idof,
                                                       const uint32_t* oline, const int32_t* row, int32_t* oc) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t h = group_vertex<G>(h0);
  if (h >= n) return;
  const int32_t D = row[h];
  if (D == 0) return;
  const int32_t x = idof[h];
  const int64_t b = rp[x], e = rp[x + 1];
  int32_t* out = oc + (int64_t)oline[h] * kTriLine;
  int32_t at = 0;
  for (int64_t k0 = b; k0 < e; k0 += G) {
    const int64_t k = k0 + lane;
    const int32_t y = k < e ? hof[ci[k]] : INT_MAX;
    const bool keep = y < h;
    const uint64_t mask = group_ballot<G>(keep);
    const int32_t p = at + (int32_t)__popcll(mask & lanes_below(lane));
    if (keep && p < D) out[p] = y + 1;
    at += (int32_t)__popcll(mask);
  }
  for (int32_t p = D + lane; p < (int32_t)tri_lines(D) * kTriLine; p += G) out[p] = 0;
}

// First h of the graph of h.
__device__ __forceinline__ int32_t tri_base(const int32_t* gid, const int64_t* vtx_off, int64_t h) {
  return gid ? (int32_t)vtx_off[gid[h]] : 0;
}

// 16-bit form of entry x of a graph that starts at base.
__device__ __forceinline__ uint16_t tri_short(int32_t x, int32_t base) {
  return x == 0 ? (uint16_t)0 : x - base <= kTriShort ? (uint16_t)(x - base) : (uint16_t)0xFFFF;
}

// Rows in decreasing order of h: up to G entries in the registers of a group
// (bitonic network over the lanes); longer ones are listed for the block kernel.
template <int G>
__global__ __launch_bounds__(256) void k_row_sort_wave(int32_t h0, int32_t n, const uint32_t* oline, const int32_t* row,
                                                       const uint32_t* wbase, const int32_t* deg, const int32_t* gid,
                                                       const int64_t* vtx_off, int32_t* oc, uint16_t* oc16,
                                                       int32_t* lu, TriLineInfo* li, int32_t* longer,
                                                       int32_t* nlonger) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t h = group_vertex<G>(h0);
  if (h >= n) return;
  const int32_t D = row[h];
  if (D == 0) return;
  const uint32_t W = tri_lines(D), l0 = oline[h];
  for (uint32_t l = lane; l < W; l += G) {
    lu[l0 + l] = (int32_t)h;
    li[l0 + l] = TriLineInfo{(int32_t)h, wbase[h], deg[h], (uint32_t)D | l << 16};
  }
  if (D > G) {
    if (lane == 0) longer[atomicAdd(nlonger, 1)] = (int32_t)h;
    return;
  }
  int32_t* out = oc + (int64_t)l0 * kTriLine;
  const bool in = lane < (int)(W * kTriLine);
  int32_t x = in ? out[lane] : 0;
  for (int k = 2; k <= G; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int32_t y = __shfl_xor(x, j, 64);
      const bool up = (lane & k) != 0;            // ascending part
      const bool low = (lane & j) == 0;
      x = (low != up) ? max(x, y) : min(x, y);
    }
  uint16_t* out16 = oc16 + (int64_t)l0 * kTriLine;
  if (in) {
    out[lane] = x;
    out16[lane] = tri_short(x, tri_base(gid, vtx_off, h));
  }
  for (int p = lane + G; p < kTriLine; p += G) out16[p] = 0;  // (of a group narrower than a line)
}

__global__ __launch_bounds__(256) void k_row_sort_block(const int32_t* longer, const int32_t* nlonger,
                                                        const uint32_t* oline, const int32_t* row,
                                                        const int32_t* gid, const int64_t* vtx_off, int32_t* oc,
                                                        uint16_t* oc16) {
  __shared__ int32_t a[kTriMaxRow];
  const int32_t cnt = *nlonger;
  for (int32_t r = blockIdx.x; r < cnt; r += gridDim.x) {
    const int32_t h = longer[r], D = row[h];
    const int64_t base = (int64_t)oline[h] * kTriLine;
    const int32_t h0 = tri_base(gid, vtx_off, h);
    int32_t P = 128;
    while (P < D) P <<= 1;
    for (int32_t k = threadIdx.x; k < P; k += 256) a[k] = k < D ? oc[base + k] : 0;
    __syncthreads();
    for (int32_t k = 2; k <= P; k <<= 1)
      for (int32_t j = k >> 1; j > 0; j >>= 1) {
        for (int32_t t = threadIdx.x; t < P / 2; t += 256) {
          const int32_t i = 2 * t - (t & (j - 1)), l = i + j;
          const int32_t p = a[i], q = a[l];
          const bool down = (i & k) == 0;  // decreasing part
          if (down ? p < q : p > q) {
            a[i] = q;
            a[l] = p;
          }
        }
        __syncthreads();
      }
    for (int32_t k = threadIdx.x; k < (int32_t)tri_lines(D) * kTriLine; k += 256) {
      const int32_t x = k < D ? a[k] : 0;
      oc[base + k] = x;
      oc16[base + k] = tri_short(x, h0);
    }
    __syncthreads();
  }
}

// Column of v in row u (decreasing), or -1.
__device__ __forceinline__ int32_t tri_find(const int32_t* r, int32_t D, int32_t v) {
  int32_t lo = 0, hi = D;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (r[mid] > v + 1) lo = mid + 1;
    else hi = mid;
  }
  return lo < D && r[lo] == v + 1 ? lo : -1;
}

__device__ __forceinline__ TriRec tri_rec(int32_t u, int32_t v, const uint32_t* oline, const uint32_t* wbase,
                                          const int32_t* row, const int32_t* oc, bool& missing) {
  TriRec r{};
  const int32_t D = row[u];
  const uint32_t l0 = oline[u];
  const int32_t i = tri_find(oc + (int64_t)l0 * kTriLine, D, v);
  missing = missing || i < 0;  // no reverse arc
  if (i < 0 || i == D - 1) return r;
  const uint32_t W = tri_lines(D);
  r.line = l0 + ((uint32_t)i >> 5);
  r.word = wbase[u] + tri_word(W, (uint32_t)i);
  r.nw = W - ((uint32_t)i >> 5);
  r.v = v;
  return r;
}

// Inclusive prefix sum over G lanes.
template <int G = 64>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, int lane) {
  for (int d = 1; d < G; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

__device__ __forceinline__ void tri_put_recs(TriRec r, uint32_t cut, TriRec* out, uint32_t p, uint32_t end) {
  for (; r.nw > 0 && p < end; ++p) {
    TriRec c = r;
    c.nw = min(r.nw, cut);
    out[p] = c;
    r.line += c.nw;
    r.word += c.nw;
    r.nw -= c.nw;
  }
}

// In-edge records of every vertex: their number and the words they hold.
__global__ __launch_bounds__(256) void k_recs_block(const BigChunk* chunks, const int32_t* ci, const int32_t* hof,
                                                    const uint32_t* oline, const uint32_t* wbase, const int32_t* row,
                                                    const int32_t* oc, const int64_t* inoff, const uint8_t* wcls,
                                                    TriRec* rec, uint32_t* inlen, int64_t* steps, int32_t* asym) {
  const BigChunk C = chunks[blockIdx.x];
  const int lane = threadIdx.x & 63;
  const uint32_t rn = (uint32_t)(inoff[C.h + 1] - inoff[C.h]);
  TriRec* out = rec + inoff[C.h];
  const uint32_t cut = wcls[C.h] ? 1 : kTriRecLines;
  unsigned long long st = 0;
  bool missing = false;
  for (int64_t k0 = C.begin; k0 < C.end; k0 += 256) {
    const int64_t k = k0 + threadIdx.x;
    const int32_t u = k < C.end ? hof[ci[k]] : -1;
    const TriRec r = u > C.h ? tri_rec(u, C.h, oline, wbase, row, oc, missing) : TriRec{};
    const uint32_t c = (r.nw + cut - 1) / cut;
    const uint32_t incl = wave_scan(c, lane), all = __shfl(incl, 63, 64);
    uint32_t base = 0;
    if (lane == 0 && all) base = atomicAdd(inlen + C.h, all);
    base = __shfl(base, 0, 64);
    tri_put_recs(r, cut, out, base + incl - c, rn);
    st += r.nw;
  }
  st = wave_sum(st);
  if (lane == 0 && st) atomicAdd(reinterpret_cast<unsigned long long*>(steps + C.h), st);
  if (__ballot(missing) && lane == 0) *asym = 1;
}

template <int G>
__global__ __launch_bounds__(256) void k_recs_wave(int32_t h0, int32_t n, const int64_t* rp, const int32_t* ci,
                                                   const int32_t* hof, const int32_t* idof, const uint32_t* oline,
                                                   const uint32_t* wbase, const int32_t* row, const int32_t* oc,
                                                   const int64_t* inoff, const uint8_t* wcls, TriRec* rec, uint32_t* inlen,
                                                   int64_t* steps, int32_t* asym) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t h = group_vertex<G>(h0);
  if (h >= n) return;
  const int32_t x = idof[h];
  const int64_t b = rp[x], e = rp[x + 1];
  const uint32_t rn = (uint32_t)(inoff[h + 1] - inoff[h]);
  TriRec* out = rec + inoff[h];
  const uint32_t cut = wcls[h] ? 1 : kTriRecLines;
  uint32_t at = 0;
  bool missing = false;
  unsigned long long st = 0;
  for (int64_t k0 = b; k0 < e; k0 += G) {
    const int64_t k = k0 + lane;
    const int32_t u = k < e ? hof[ci[k]] : -1;
    const TriRec r = u > (int32_t)h ? tri_rec(u, (int32_t)h, oline, wbase, row, oc, missing) : TriRec{};
    const uint32_t c = (r.nw + cut - 1) / cut;
    const uint32_t incl = wave_scan<G>(c, lane);
    tri_put_recs(r, cut, out, at + incl - c, rn);
    at += __shfl(incl, (threadIdx.x & 63) | (G - 1), 64);
    st += r.nw;
  }
  st = group_sum<G>(st);
  if (lane == 0) {
    inlen[h] = min(at, rn);
    steps[h] = (int64_t)st;
  }
  if (G < 64)  // k_tri_few goes through all of them
    for (uint32_t p = at + lane; p < rn; p += G) out[p] = TriRec{};
  if (missing) *asym = 1;
}

// Work of every vertex: jobs of the block kernel, or a place in the wave
// kernel's list (from `few` on, none); the sum of all words and the longest
// hash-table row.
__global__ void k_job_counts(int32_t n, int32_t few, const int32_t* gid, const int64_t* vtx_off, const int32_t* row,
                             const uint8_t* wcls, const uint32_t* inlen, const int64_t* steps, int64_t* njob,
                             int64_t* nwave, uint32_t part, unsigned long long* total, int32_t* max_hash) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  unsigned long long st = 0;
  int32_t most = 0;
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h <= n; h += stride) {
    int64_t j = 0, w = 0;
    if (h < n && steps[h] > 0) {
      st += (unsigned long long)steps[h];
      if (h >= few) {
      } else if (wcls[h]) {
        w = (inlen[h] + part - 1) / part;
      } else {
        j = (inlen[h] + kTriJob - 1) / kTriJob;
        if (h - tri_base(gid, vtx_off, h) >= kTriShort) most = max(most, row[h]);
      }
    }
    njob[h] = j;
    nwave[h] = w;
  }
  st = wave_sum(st);
  for (int d = 32; d >= 1; d >>= 1) most = max(most, __shfl_xor(most, d, 64));
  if ((threadIdx.x & 63) == 0) {
    if (st) atomicAdd(total, st);
    if (most > 0) atomicMax(max_hash, most);
  }
}

__global__ void k_job_fill(int32_t n, const int64_t* inoff, const uint32_t* inlen, const uint32_t* oline, const int32_t* row,
                           const int64_t* job_at, const int64_t* wave_at, uint32_t part, TriJob* job, TriWave* wrow) {
  const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= n) return;
  const int64_t j0 = job_at[h], nj = job_at[h + 1] - j0;
  const uint32_t r0 = (uint32_t)inoff[h], r1 = r0 + inlen[h];
  const int64_t w0 = wave_at[h], nw = wave_at[h + 1] - w0;
  for (int64_t j = 0; j < nw; ++j) {
    const uint32_t beg = r0 + (uint32_t)j * part, cnt = min(part, r1 - beg);
    wrow[w0 + j] = TriWave{(int32_t)h, oline[h], beg, (uint32_t)row[h] | cnt << 8 | (nw == 1 ? kTriWaveSingle : 0)};
  }
  for (int64_t j = 0; j < nj; ++j) {
    TriJob J;
    J.v = (int32_t)h;
    J.rbeg = r0 + (uint32_t)(j * kTriJob);
    J.rcnt = min((uint32_t)kTriJob, r1 - J.rbeg);
    J.single = nj == 1;
    job[j0 + j] = J;
  }
}

// Edges per degree bucket (lane per entry, smaller side = the row's vertex).
__global__ __launch_bounds__(256) void k_tri_buckets(int64_t lines, const int32_t* lu, const int32_t* oc,
                                                     const int32_t* deg, unsigned long long* out) {
  __shared__ uint32_t c[kNumBuckets];
  if (threadIdx.x < kNumBuckets) c[threadIdx.x] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < lines * kTriLine; i += stride) {
    const int32_t x = oc[i] - 1;
    int b = -1;
    if (x >= 0) {
      b = bucket_of(deg[lu[i >> 5]]);
      if (b == 5 && deg[x] > kHubMinDegree) b = 6;
    }
    for (int k = 0; k < kNumBuckets; ++k) {
      const uint64_t m = __ballot(b == k);
      if (m && (threadIdx.x & 63) == 0) atomicAdd(&c[k], (uint32_t)__popcll(m));
    }
  }
  __syncthreads();
  if (threadIdx.x < kNumBuckets && c[threadIdx.x]) atomicAdd(out + threadIdx.x, (unsigned long long)c[threadIdx.x]);
}

// ---------------------------------------------------------------------------
// Counting

// w of lane `to` = x (x and `to` uniform).  The write-lane instruction has no
// builtin, so its intrinsic is declared by name.  Not an asm statement: x comes
// from a compare, and a vector instruction may read a compare's scalar result
// only two wait states later, which the compiler sees to only for instructions
// that it can see (as asm it directly followed the compare in 24 places).
__device__ int32_t write_lane(int32_t x, int32_t to, int32_t old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ void set_lane(uint32_t& w, uint32_t x, const int to) {
  w = (uint32_t)write_lane((int32_t)x, to, (int32_t)w);
}

// Accesses through a buffer descriptor that ends where the record ends: loads
// past it give 0 (no entry) and stores nothing, without touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_upto(const void* base, uint32_t end) {
  constexpr int kFlags = 0x00027000;  // raw 32-bit data
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)end, kFlags);
}
__device__ __forceinline__ uint16_t buffer_entry(const uint16_t*, __amdgpu_buffer_rsrc_t b, uint32_t at) {
  return __builtin_amdgcn_raw_buffer_load_b16(b, (int)at, 0, 0);
}
__device__ __forceinline__ uint32_t buffer_entry(const uint32_t*, __amdgpu_buffer_rsrc_t b, uint32_t at) {
  return __builtin_amdgcn_raw_buffer_load_b32(b, (int)at, 0, 0);
}

using LdsCounter = __attribute__((address_space(3))) int32_t;

// Columns of one job's in-edges through a lookup: find(x) is the LDS address
// of x's counter, or 0.  A wave takes a run of the records, one at a time (up
// to 8 lines) and 64 columns a step, so that addresses and loop are scalar and
// a ballot is two words of bits.  Each lane works out the offsets of one record
// of 64, read back one after the other: scalar instructions, of which a compute
// unit issues one a cycle for all its waves, bounded the loop when every record
// was decoded in scalar code.  The next three records are loaded while one is
// looked up (R-MAT scale 22: 6.6 ms with one of them under way, 6.25 with three;
// scale 17: 95 and 80 us); all four loads are always issued, since a load under a
// branch would make the compiler wait for every load in flight.  At scale 22
// 22.8 GB are then read past the L2s (13 % hits) and 3.2 written, 3.9 TB/s of the
// 4.9 of a large copy, with the vector units busy 59 % of the cycles and the LDS 36 %.
// Columns up to v's own are in no table of v (h(w) >= h(v)) and need no mask.
template <typename E, typename F>
__device__ __forceinline__ void tri_stream(const E* __restrict__ cols, const TriRec* __restrict__ rec, uint32_t cnt,
                                           uint32_t wave, int lane, uint32_t* __restrict__ bits, F find) {
  static_assert(kTriRecLines == 8, "four steps of two lines");
  constexpr uint32_t kLineBytes = kTriLine * sizeof(E), kStep = 64 * sizeof(E);
  struct Cols {
    E c0, c1, c2, c3;  // (named: an array is kept as one vector, which waits for all of it)
  };
  // (two clamped ends: written as a saturating difference, the compiler drops
  // the saturation of the scalar subtraction)
  const uint32_t per = (cnt + kTriBlock / 64 - 1) / (kTriBlock / 64);
  const uint32_t first = min(wave * per, cnt), n = min(wave * per + per, cnt) - first;
  const uint32_t at = (uint32_t)lane * sizeof(E), wat = (uint32_t)lane * 4;
  for (uint32_t b0 = 0; b0 < n; b0 += kTriBatch) {
    const uint32_t nb = min((uint32_t)kTriBatch, n - b0);
    const TriRec r = (uint32_t)lane < nb ? rec[first + b0 + lane] : TriRec{};
    // 16-bit entries: byte offsets of the record; 32-bit ones, which would pass
    // 32 bits on the largest graphs: its line, and its length
    const int off = (int)(sizeof(E) == 2 ? r.line * kLineBytes : r.line);
    const int end = (int)((sizeof(E) == 2 ? r.line + r.nw : r.nw) * kLineBytes);
    const int woff = (int)(r.word * 4), wend = (int)((r.word + r.nw) * 4);
    auto load = [&](Cols& y, uint32_t i) {  // i >= nb: a record of no lines
      uint32_t o = at, upto = (uint32_t)__builtin_amdgcn_readlane(end, (int)i);
      const E* from = cols;
      if (sizeof(E) == 2) o += (uint32_t)__builtin_amdgcn_readlane(off, (int)i);
      else from += (uint64_t)(uint32_t)__builtin_amdgcn_readlane(off, (int)i) * kTriLine;
      const __amdgpu_buffer_rsrc_t b = buffer_upto(from, upto);
      y.c0 = buffer_entry(cols, b, o);
      y.c1 = buffer_entry(cols, b, o + kStep);
      y.c2 = buffer_entry(cols, b, o + 2 * kStep);
      y.c3 = buffer_entry(cols, b, o + 3 * kStep);
    };
    auto look = [&](const Cols& x, uint32_t i) {
      const uint32_t so = (uint32_t)__builtin_amdgcn_readlane(woff, (int)i);
      const uint32_t se = (uint32_t)__builtin_amdgcn_readlane(wend, (int)i);
      const uint32_t left = se - so;  // bytes of bits: 4 per line
      uint32_t w = 0;
      auto step = [&](E col, auto k) {
        constexpr int kAt = decltype(k)::value;
        const uint32_t place = find(col);
        const bool hit = place != 0;
        const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
        if (hit) __hip_atomic_fetch_add((LdsCounter*)(uintptr_t)place, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        set_lane(w, (uint32_t)m, 2 * kAt);
        set_lane(w, (uint32_t)(m >> 32), 2 * kAt + 1);
      };
      if (left > 0) {
        step(x.c0, std::integral_constant<int, 0>{});
        if (left > 8) {
          step(x.c1, std::integral_constant<int, 1>{});
          if (left > 16) {
            step(x.c2, std::integral_constant<int, 2>{});
            if (left > 24) step(x.c3, std::integral_constant<int, 3>{});
          }
        }
      }
      __builtin_amdgcn_raw_buffer_store_b32(w, buffer_upto(bits, se), (int)(wat + so), 0, 0);
    };
    Cols x, y, z, u;
    load(x, 0);
    load(y, 1);
    load(z, 2);
    for (uint32_t i = 0; i < nb; i += 4) {
      load(u, i + 3);
      look(x, i);
      load(x, i + 4);
      look(y, i + 1);
      load(y, i + 5);
      look(z, i + 2);
      load(z, i + 6);
      look(u, i + 3);
    }
  }
}

__host__ __device__ inline uint32_t tri_hash_slots(int32_t D) {
  uint32_t s = 64;
  while (s < 2u * (uint32_t)D) s <<= 1;
  return s;
}

__device__ __forceinline__ uint32_t tri_hash(int32_t x) { return (uint32_t)x * 0x9E3779B1u >> 12; }

// One job: row v into LDS, its in-edges streamed past it.  Three tables:
//   h(v) < kTriDirect  16 bits per h below h(v): the address of the entry's counter;
//   h(v) < kTriShort   a bit per h and, per 32 of them, the places before;
//   above              a hash set of the entries, linear probing, at most half full.
// The first two read the 16-bit columns.  Block-uniform choice.
__device__ __forceinline__ void tri_job(const TriJob J, int32_t* tri_lds, const TriRec* __restrict__ rec,
                                        const int32_t* __restrict__ row, const uint32_t* __restrict__ oline,
                                        const int32_t* __restrict__ gid, const int64_t* __restrict__ vtx_off,
                                        const int32_t* __restrict__ oc, const uint16_t* __restrict__ oc16,
                                        uint32_t* __restrict__ bits, int32_t* __restrict__ cnt, uint32_t acc_cap) {
  const int32_t D = row[J.v], h0 = tri_base(gid, vtx_off, J.v), v = J.v - h0;  // v within its graph
  const int64_t base = (int64_t)oline[J.v] * kTriLine;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds = (uint32_t)(uintptr_t)(LdsCounter*)tri_lds;  // LDS address of the counters
  const TriRec* recs = rec + J.rbeg;
  auto put = [&](int32_t j, int32_t c) {
    if (!c) return;
    if (J.single) cnt[base + j] = c;
    else atomicAdd(cnt + base + j, c);
  };
  int32_t* acc = tri_lds;
  int32_t* tab = tri_lds + acc_cap;
  if (v < kTriShort) {
    for (int32_t k = tid; k <= D; k += kTriBlock) acc[k] = 0;
    if (v < kTriDirect) {
      uint16_t* t16 = reinterpret_cast<uint16_t*>(tab);
      for (int32_t k = tid; k < (v + 1) / 8 + 1; k += kTriBlock)
        reinterpret_cast<int4*>(tab)[k] = make_int4(0, 0, 0, 0);
      __syncthreads();
      static_assert(4 * (kTriMaxRow + 1) <= 0xFFFF, "addresses in 16 bits");
      for (int32_t j = tid; j < D; j += kTriBlock) t16[oc[base + j] - h0] = (uint16_t)(lds + 4 * (j + 1));
      __syncthreads();
      // entry v + 1 (and 0, no entry) stays 0
      tri_stream(oc16, recs, J.rcnt, wave, lane, bits, [&](uint16_t x) -> uint32_t {
        uint32_t p = t16[min(x, (uint16_t)(v + 1))];
        asm("" : "+v"(p));  // a 32-bit value from here on (the load extends it)
        return p;
      });
      __syncthreads();
      for (int32_t j = tid; j < D; j += kTriBlock) put(j, acc[j + 1]);
    } else {
      uint2* tb = reinterpret_cast<uint2*>(tab);
      const int32_t nt = ((v + 1) >> 5) + 1;
      for (int32_t k = tid; k < nt; k += kTriBlock) tb[k] = make_uint2(0, 0);
      __syncthreads();
      for (int32_t j = tid; j < D; j += kTriBlock) {
        const int32_t x = oc[base + j] - h0;
        atomicOr(&tb[x >> 5].x, 1u << (x & 31));
      }
      __syncthreads();
      // entries before each word: one wave, 64 words a step
      if (tid < 64) {
        uint32_t before = 0;
        for (int32_t k0 = 0; k0 < nt; k0 += 64) {
          const int32_t k = k0 + lane;
          const uint32_t c = k < nt ? (uint32_t)__popc(tb[k].x) : 0;
          uint32_t incl = c;
          for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
          }
          if (k < nt) tb[k].y = before + incl - c;
          before += __shfl(incl, 63, 64);
        }
      }
      __syncthreads();
      auto find = [&](uint16_t x) -> uint32_t {
        const uint32_t o = min(x, (uint16_t)(v + 1));  // bits 0 (no entry) and v + 1 are not set
        const uint2 t = tb[o >> 5];
        const uint32_t upto = t.x << (~o & 31);
        return (int32_t)upto < 0 ? lds + 4 * (t.y + (uint32_t)__popc(upto)) : 0;
      };
      tri_stream(oc16, recs, J.rcnt, wave, lane, bits, find);
      __syncthreads();
      for (int32_t j = tid; j < D; j += kTriBlock) put(j, acc[(find((uint16_t)(oc[base + j] - h0)) - lds) / 4]);
    }
  } else {
    const uint32_t slots = tri_hash_slots(D), mask = slots - 1;
    int32_t* key = tri_lds;
    int32_t* hits = tri_lds + slots;
    for (uint32_t k = tid; k < slots; k += kTriBlock) {
      key[k] = -1;
      hits[k] = 0;
    }
    __syncthreads();
    for (int32_t j = tid; j < D; j += kTriBlock) {
      const int32_t x = oc[base + j];
      uint32_t t = tri_hash(x) & mask;
      while (atomicCAS(key + t, -1, x) != -1) t = (t + 1) & mask;
    }
    __syncthreads();
    auto find = [&](uint32_t x) -> uint32_t {
      if (x - 1 >= (uint32_t)J.v) return 0;  // no entry included
      uint32_t t = tri_hash((int32_t)x) & mask;
      while (true) {
        const int32_t y = key[t];
        if (y == (int32_t)x) return lds + 4 * (slots + t);
        if (y == -1) return 0;
        t = (t + 1) & mask;
      }
    };
    tri_stream(reinterpret_cast<const uint32_t*>(oc), recs, J.rcnt, wave, lane, bits, find);
    __syncthreads();
    for (int32_t j = tid; j < D; j += kTriBlock) put(j, tri_lds[(find((uint32_t)oc[base + j]) - lds) / 4]);
  }
}

// Vertices with a short row and few in-edges, a wave each or per part; a record is one
// line, and each half of the wave takes every other one.  Bound by vector
// instructions (batch of 300 graphs: 0.8 of 1.16 ms when every line's place was
// worked out here and every lookup could take several probes), so: records of
// one line, offsets read back from the lane that loaded the record, the bits of
// four steps stored by eight lanes at once, and for rows up to 40 entries (256
// slots) a hash that is changed until the row has no collision, after which a
// lookup is one probe (batch of 300 graphs: 0.77 ms).
template <typename E>
__device__ __forceinline__ void tri_row(const TriWave V, int32_t* key, const TriRec* __restrict__ rec,
                                        const E* __restrict__ cols, int64_t lines, uint32_t* __restrict__ bits,
                                        int32_t* __restrict__ cnt) {
  constexpr uint32_t kMask = kTriWaveSlots - 1;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  const int lane = threadIdx.x & 63, half = lane >> 5, sub = lane & 31;
  int32_t* hit = key + kTriWaveSlots;
  const uint32_t D = V.shape & 0xFFu, rc = (V.shape & ~kTriWaveSingle) >> 8;
  const int64_t base = (int64_t)V.line * kTriLine;
  const TriRec* recs = rec + V.rbeg;
  const uint32_t e0 = (uint32_t)lane < D ? cols[base + lane] : 0;
  const uint32_t e1 = D > 64 && (uint32_t)lane + 64 < D ? cols[base + 64 + lane] : 0;
  TriRec r = (uint32_t)lane < rc ? recs[lane] : TriRec{kNone, 0, 0, 0};
  static_assert(kTriWaveSlots == 1 << 8 && kTriWaveRow <= 128, "four slots per lane, two entries per lane");
  uint32_t shift = 8, t0 = 0, t1 = 0;
  // one probe per lookup, or (the neighbours of hubs are runs of ids, which the
  // folded hash would put side by side) a scattering hash with linear probing
  bool single = D <= 40;
  auto hash = [&](uint32_t x) -> uint32_t {
    return single ? (x ^ (x >> shift)) & kMask : x * 0x9E3779B1u >> 24;
  };
  reinterpret_cast<int4*>(hit)[lane] = make_int4(0, 0, 0, 0);
  for (int attempt = 0;; ++attempt) {
    reinterpret_cast<int4*>(key)[lane] = make_int4(-1, -1, -1, -1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    t0 = hash(e0);
    t1 = hash(e1);
    bool ok = e0 == 0 || atomicCAS(key + t0, -1, (int32_t)e0) == -1;
    bool ok1 = e1 == 0 || atomicCAS(key + t1, -1, (int32_t)e1) == -1;
    if (!__ballot(!(ok && ok1))) break;
    if (single) {
      shift = attempt == 0 ? 5 : attempt == 1 ? 3 : 10;
      single = attempt < 3;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      continue;
    }
    while (!ok) {
      t0 = (t0 + 1) & kMask;
      ok = atomicCAS(key + t0, -1, (int32_t)e0) == -1;
    }
    while (!ok1) {
      t1 = (t1 + 1) & kMask;
      ok1 = atomicCAS(key + t1, -1, (int32_t)e1) == -1;
    }
    break;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  struct Group {
    E x0, x1, x2, x3;
  };
  const __amdgpu_buffer_rsrc_t all = buffer_upto(cols, (uint32_t)(lines * kTriLine * 2));  // (16-bit entries)
  for (uint32_t b0 = 0; b0 < rc; b0 += 64) {
    if (b0) r = b0 + lane < rc ? recs[b0 + lane] : TriRec{kNone, 0, 0, 0};
    const uint32_t nb = min(64u, rc - b0);
    // 16-bit entries: the byte offset (past the end for no record); else the line
    const int where = (int)(sizeof(E) == 2 ? (r.line == kNone ? kNone : r.line * (kTriLine * 2)) : r.line);
    auto entry = [&](uint32_t k) -> E {
      const uint32_t o = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((k + half) * 4), where);
      if (sizeof(E) == 2) return (E)buffer_entry((const uint16_t*)nullptr, all, o == kNone ? o : o + 2 * sub);
      return o == kNone ? (E)0 : cols[(int64_t)o * kTriLine + sub];
    };
    auto load = [&](Group& g, uint32_t k) {
      g.x0 = entry(k);
      g.x1 = entry(k + 2);
      g.x2 = entry(k + 4);
      g.x3 = entry(k + 6);
    };
    auto look = [&](const Group& g, uint32_t k) {
      uint32_t w = 0;
      auto step = [&](E x, auto at) {
        constexpr int kAt = decltype(at)::value;
        uint32_t t = hash(x);
        int32_t y = key[t];
        if (!single) {
          while (y != (int32_t)x && y != -1) {
            t = (t + 1) & kMask;
            y = key[t];
          }
        }
        const bool found = y == (int32_t)x;  // 0, no entry, is in no table
        if (found) atomicAdd(hit + t, 1);
        const uint64_t m = __builtin_amdgcn_ballot_w64(found);
        set_lane(w, (uint32_t)m, 2 * kAt);
        set_lane(w, (uint32_t)(m >> 32), 2 * kAt + 1);
      };
      step(g.x0, std::integral_constant<int, 0>{});
      step(g.x1, std::integral_constant<int, 1>{});
      step(g.x2, std::integral_constant<int, 2>{});
      step(g.x3, std::integral_constant<int, 3>{});
      const uint32_t to = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((k + lane) * 4), (int)r.word);
      if (lane < 8 && k + lane < nb) bits[to] = w;
    };
    Group g, h;
    load(g, 0);
    for (uint32_t k = 0; k < nb; k += 16) {
      if (k + 8 < nb) load(h, k + 8);
      look(g, k);
      if (k + 8 >= nb) break;
      if (k + 16 < nb) load(g, k + 16);
      look(h, k + 8);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  auto put = [&](int64_t at, int32_t c) {
    if (V.shape & kTriWaveSingle) cnt[at] = c;
    else if (c) atomicAdd(cnt + at, c);
  };
  if (e0) put(base + lane, hit[t0]);
  if (e1) put(base + 64 + lane, hit[t1]);
}

// Rows of a graph without jobs, four waves a block (in blocks of eight, as
// below, 300 planted graphs take 0.81 instead of 0.77 ms).
template <typename E>
__global__ __launch_bounds__(256) void k_tri_wave(int64_t nrow, const TriWave* __restrict__ wrow,
                                                  const TriRec* __restrict__ rec, const E* __restrict__ cols,
                                                  int64_t lines, uint32_t* __restrict__ bits,
                                                  int32_t* __restrict__ cnt) {
  __shared__ __align__(16) int32_t sets[4][2 * kTriWaveSlots];
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i < nrow) tri_row(wrow[i], sets[threadIdx.x >> 6], rec, cols, lines, bits, cnt);
}

// Records of vertices of at most kNarrowRow neighbours, one per thread: row u
// and row v have a line and at most 8 entries each.  In a wave per vertex nearly
// all lanes were idle or on padding, and one chain of loads was under way: 3.05 ms
// on a triangulated grid of 9 million vertices (26 million records), now 0.88, at
// 3.7 TB/s for the 128 bytes a record reads and writes; 0.62 and 0.16 on a
// road-like grid of 4 million.
static_assert(kNarrowRow == 8, "two loads of four entries");
__global__ __launch_bounds__(256) void k_tri_few(int64_t few, const TriRec* __restrict__ rec,
                                                 const int32_t* __restrict__ row, const uint32_t* __restrict__ oline,
                                                 const int32_t* __restrict__ oc, uint32_t* __restrict__ bits,
                                                 int32_t* __restrict__ cnt) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= few) return;
  const TriRec r = rec[i];
  if (r.nw == 0) return;
  const int32_t D = row[r.v];
  const int64_t base = (int64_t)oline[r.v] * kTriLine;
  const int4* mine = reinterpret_cast<const int4*>(oc + base);
  const int4* theirs = reinterpret_cast<const int4*>(oc + (int64_t)r.line * kTriLine);
  const int4 none = make_int4(0, 0, 0, 0);
  const int4 a0 = theirs[0], a1 = theirs[1], b0 = D > 0 ? mine[0] : none, b1 = D > 4 ? mine[1] : none;
  const int32_t b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
  uint32_t w = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (b[j] == 0) continue;  // no entry
    const uint32_t hit = (a0.x == b[j] ? 1u : 0u) | (a0.y == b[j] ? 2u : 0u) | (a0.z == b[j] ? 4u : 0u) |
                         (a0.w == b[j] ? 8u : 0u) | (a1.x == b[j] ? 16u : 0u) | (a1.y == b[j] ? 32u : 0u) |
                         (a1.z == b[j] ? 64u : 0u) | (a1.w == b[j] ? 128u : 0u);
    if (hit) atomicAdd(cnt + base + j, 1);
    w |= hit;
  }
  bits[r.word] = w;
}

// Jobs and waves' rows in one launch, spread evenly over it: `ratio` is the
// share of the blocks that take a job, in 2^-32.  The jobs wait for memory and
// the rows for vector instructions, so they run well side by side, and on a small
// graph neither fills the chip (R-MAT scale 14: 21 and 18 us one after the other,
// 24 together; scale 17: 79 and 37, 109; scale 22 the same within 1 %).
template <typename E>
__global__ __launch_bounds__(kTriBlock) __attribute__((amdgpu_waves_per_eu(8, 8)))
void k_tri_count(uint64_t ratio, const TriJob* __restrict__ jobs, int64_t nrow, const TriWave* __restrict__ wrow,
                 const TriRec* __restrict__ rec, const int32_t* __restrict__ row, const uint32_t* __restrict__ oline,
                 const int32_t* __restrict__ gid, const int64_t* __restrict__ vtx_off,
                 const int32_t* __restrict__ oc, const uint16_t* __restrict__ oc16, int64_t lines,
                 uint32_t* __restrict__ bits, int32_t* __restrict__ cnt, uint32_t acc_cap) {
  extern __shared__ __align__(16) int32_t tri_lds[];
  const uint32_t before = (uint32_t)((uint64_t)blockIdx.x * ratio >> 32);  // blocks before this one with a job
  if ((uint32_t)(((uint64_t)blockIdx.x + 1) * ratio >> 32) > before) {
    tri_job(jobs[before], tri_lds, rec, row, oline, gid, vtx_off, oc, oc16, bits, cnt, acc_cap);
    return;
  }
  const uint32_t wave = threadIdx.x >> 6;
  const int64_t i = (int64_t)(blockIdx.x - before) * (kTriBlock / 64) + wave;
  if (i >= nrow) return;
  if constexpr (sizeof(E) == 2)
    tri_row(wrow[i], tri_lds + wave * 2 * kTriWaveSlots, rec, oc16, lines, bits, cnt);
  else
    tri_row(wrow[i], tri_lds + wave * 2 * kTriWaveSlots, rec, reinterpret_cast<const uint32_t*>(oc), lines, bits, cnt);
}

// ---------------------------------------------------------------------------
// From counts to clusters

__global__ void k_tri_init(int64_t ncnt4, int4* cnt, int32_t n, int32_t* lower, int32_t* parent, int32_t* label,
                           uint8_t* role, int32_t* flag) {
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = i0; i < ncnt4; i += stride) cnt[i] = make_int4(0, 0, 0, 0);
  if (i0 == 0) *flag = 0;
  if (!lower) return;
  for (int64_t u = i0; u < n; u += stride) {
    lower[u] = 1;  // u itself is in N_eps[u]
    parent[u] = (int32_t)u;
    label[u] = INT_MAX;
    role[u] = 0;
  }
}

__device__ __forceinline__ int32_t tri_mu(const TriArgs& a, int64_t h) { return a.gid ? a.gmu[a.gid[h]] : a.mu; }

// x of the lane whose number differs by kXor inside the half wave.
template <int kXor>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  if constexpr (kXor == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1 /* quad 1,0,3,2 */, 0xF, 0xF, true);
  if constexpr (kXor == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E /* quad 2,3,0,1 */, 0xF, 0xF, true);
  if constexpr (kXor == 4) {  // 7 - lane of eight, then 3 - lane of four
    const int y = __builtin_amdgcn_update_dpp(0, (int)x, 0x141 /* row_half_mirror */, 0xF, 0xF, true);
    return (uint32_t)__builtin_amdgcn_update_dpp(0, y, 0x1B /* quad 3,2,1,0 */, 0xF, 0xF, true);
  }
  if constexpr (kXor == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128 /* row_ror:8 */, 0xF, 0xF, true);
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x401F /* lane ^ 16 */);
}

// 32 x 32 bits across the lanes of a half wave: lane j's word becomes column j.
template <int kStep>
__device__ __forceinline__ uint32_t tri_exchange(uint32_t w, int sub, uint32_t m) {
  const uint32_t y = lane_xor<kStep>(w);
  return (sub & kStep) ? (w & ~m) | ((y & ~m) >> kStep) : (w & m) | ((y & m) << kStep);
}
__device__ __forceinline__ uint32_t tri_transpose(uint32_t w, int sub) {
  w = tri_exchange<16>(w, sub, 0x0000FFFFu);
  w = tri_exchange<8>(w, sub, 0x00FF00FFu);
  w = tri_exchange<4>(w, sub, 0x0F0F0F0Fu);
  w = tri_exchange<2>(w, sub, 0x33333333u);
  return tri_exchange<1>(w, sub, 0x55555555u);
}

// Similar entries of line t (half wave), counted on both endpoints.
__device__ __forceinline__ void tri_mark(int64_t t, int sub, const TriLineInfo& L, int32_t x, int32_t dx,
                                         int32_t closed, TriArgs& a, uint32_t* simw, int32_t* lower) {
  if (a.gid) {
    const int32_t g = a.gid[L.u];
    a.p = a.gp[g];
    a.q = a.gq[g];
  }
  bool sim = false;
  if (x >= 0) {
    const uint64_t ab = ((uint64_t)L.deg + 1) * ((uint64_t)dx + 1);
    const uint64_t cq = (uint64_t)closed * a.q;
    sim = cq * cq >= (a.p * a.p) * ab;
  }
  const uint64_t m = __ballot(sim);
  const uint32_t word = (threadIdx.x & 32) ? (uint32_t)(m >> 32) : (uint32_t)m;
  if (sub == 0) {
    simw[t] = word;
    if (word) atomicAdd(lower + L.u, (int32_t)__popc(word));
  }
  if (sim) atomicAdd(lower + x, 1);
}

// Block of lines that block b of nb takes.  In a batch the blocks of an XCD (every
// eighth) take consecutive ones, so that a graph's vertices are read through one
// L2 (300 graphs: k_tri_close 380 -> 358 us, k_tri_hook 237 -> 166; k_tri_link and
// k_tri_attach, which wait for atomics, and k_tri_wave got slower).  Of a single
// graph that would put all the long rows on the first XCD.
__device__ __forceinline__ int64_t line_block(int64_t b, int64_t nb, const TriArgs& a) {
  const int64_t per = nb >> 3;
  return a.gid && b < per * 8 ? (b & 7) * per + (b >> 3) : b;
}

// One line per half wave: closed counts of its entries, and with eps the
// similar ones.
template <bool kEps>
__global__ __launch_bounds__(256) void k_tri_close(int64_t lines, const TriLineInfo* __restrict__ li,
                                                   const int32_t* __restrict__ deg, const int32_t* __restrict__ oc,
                                                   const uint32_t* __restrict__ bits, int32_t* __restrict__ cnt,
                                                   TriArgs a, uint32_t* __restrict__ simw,
                                                   int32_t* __restrict__ lower) {
  const int64_t t = line_block(blockIdx.x, gridDim.x, a) * 8 + (threadIdx.x >> 5);
  if (t >= lines) return;
  const int sub = threadIdx.x & 31;
  const TriLineInfo L = li[t];
  const int32_t x = oc[t * kTriLine + sub] - 1;
  int32_t closed = cnt[t * kTriLine + sub] + 2;
  const int32_t D = (int32_t)(L.shape & 0xFFFFu);
  const uint32_t W = tri_lines(D), c = L.shape >> 16;
  const int32_t i = (int32_t)(c * kTriLine) + sub;
  // the row's own bits (the last column has none after it and was not written)
  const uint32_t* mine = bits + L.wbase + tri_word(W, (uint32_t)i);
  const uint32_t own = i < D - 1 ? *mine : 0;
  if (i < D - 1)
    for (uint32_t k = 1; k < W - c; ++k) closed += __popc(mine[k]);
  const int32_t dx = kEps && x >= 0 ? deg[x] : 0;
  // the bits of its column
  for (uint32_t b = 0; b < c; ++b) {
    const uint32_t k = b * kTriLine + sub;
    closed += __popc(tri_transpose(bits[L.wbase + tri_word(W, k) + (c - b)], sub));
  }
  closed += __popc(own) + __popc(tri_transpose(own, sub));
  if (!kEps) {
    cnt[t * kTriLine + sub] = closed;
    return;
  }
  tri_mark(t, sub, L, x, dx, closed, a, simw, lower);
}

// The same from closed counts already in cnt.
__global__ __launch_bounds__(256) void k_tri_threshold(int64_t lines, const TriLineInfo* __restrict__ li,
                                                       const int32_t* __restrict__ deg,
                                                       const int32_t* __restrict__ oc,
                                                       const int32_t* __restrict__ cnt, TriArgs a,
                                                       uint32_t* __restrict__ simw, int32_t* __restrict__ lower) {
  const int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 5;
  if (t >= lines) return;
  const int sub = threadIdx.x & 31;
  const int32_t x = oc[t * kTriLine + sub] - 1;
  tri_mark(t, sub, li[t], x, x >= 0 ? deg[x] : 0, cnt[t * kTriLine + sub], a, simw, lower);
}

// A parent as the caches have it: some ancestor, maybe not the newest.
__device__ __forceinline__ int32_t ld_near(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Minimum over a half wave.
__device__ __forceinline__ int32_t half_min(int32_t x) {
  x = min(x, (int32_t)lane_xor<16>((uint32_t)x));
  x = min(x, (int32_t)lane_xor<8>((uint32_t)x));
  x = min(x, (int32_t)lane_xor<4>((uint32_t)x));
  x = min(x, (int32_t)lane_xor<2>((uint32_t)x));
  return min(x, (int32_t)lane_xor<1>((uint32_t)x));
}

// First step of the clustering: every core points at the least core id that a
// line joins it to.  A parent is a smaller core of the same cluster, so this is
// a forest, got with one atomicMin per similar entry at most and no retries,
// and in a dense cluster it leaves few roots for k_tri_hook, where unions of
// single edges from the start compete for the same roots.
// Sets the flag that lets the later kernels run: a core has a similar entry.
__global__ __launch_bounds__(256) void k_tri_link(int64_t lines, const int32_t* __restrict__ lu,
                                                  const int32_t* __restrict__ oc, const uint32_t* __restrict__ simw,
                                                  const int32_t* __restrict__ lower, const int32_t* __restrict__ idof,
                                                  TriArgs a_, int32_t* parent, int32_t* __restrict__ flag) {
  const int sub = threadIdx.x & 31;
  const int64_t stride = (int64_t)gridDim.x * 8;
  bool cores = false;
  for (int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 5; t < lines; t += stride) {
    const uint32_t w = simw[t];
    if (!w) continue;
    const int32_t u = lu[t], mu = tri_mu(a_, u);
    const int32_t x = oc[t * kTriLine + sub] - 1;
    const bool in = ((w >> sub) & 1u) && lower[x] >= mu;
    cores = cores || in;
    if (lower[u] < mu) continue;
    cores = true;
    const int32_t a = idof[u], b = in ? idof[x] : a;
    const int32_t least = half_min(min(a, b));
    if (in && least < b && ld_near(parent + b) > least) atomicMin(parent + b, least);
    if (sub == 0 && least < a && ld_near(parent + a) > least) atomicMin(parent + a, least);
  }
  if (__ballot(cores) && (threadIdx.x & 63) == 0) *flag = 1;
}

__global__ void k_tri_compress(int32_t n, int32_t* parent, const int32_t* __restrict__ flag) {
  if (!*flag) return;
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const int32_t p = ld_i32(parent + x);
  if (p == (int32_t)x) return;
  const int32_t r = uf_find(parent, p);
  if (r != p) st_i32(parent + x, r);
}

// The rest of the unions: the roots that a line's entries found are hooked
// below the least of them, each by one lane.
__global__ __launch_bounds__(256) void k_tri_hook(int64_t lines, const int32_t* __restrict__ lu,
                                                  const int32_t* __restrict__ oc, const uint32_t* __restrict__ simw,
                                                  const int32_t* __restrict__ lower, const int32_t* __restrict__ idof,
                                                  TriArgs a_, int32_t* parent, const int32_t* __restrict__ flag) {
  if (!*flag) return;
  const int lane = threadIdx.x & 63, half = lane >> 5, sub = lane & 31;
  const int64_t blocks = (lines + 7) >> 3;
  for (int64_t k = blockIdx.x; k < blocks; k += gridDim.x) {
    const int64_t t = line_block(k, blocks, a_) * 8 + (threadIdx.x >> 5);
    const uint32_t w = t < lines ? simw[t] : 0;
    if (!w) continue;
    const int32_t u = lu[t], mu = tri_mu(a_, u);
    if (lower[u] < mu) continue;
    const int32_t x = oc[t * kTriLine + sub] - 1;
    const bool in = ((w >> sub) & 1u) && lower[x] >= mu;
    const int32_t a = idof[u], b = in ? idof[x] : a;
    // most lines are one tree already
    const int32_t na = ld_near(parent + a), nb = in ? ld_near(parent + b) : na;
    const uint64_t differ = __ballot(na != nb);
    if (!(half ? (uint32_t)(differ >> 32) : (uint32_t)differ)) continue;
    int32_t ra = uf_find(parent, na);
    int32_t rb = in ? uf_find(parent, nb) : ra;
    while (true) {
      const int32_t least = half_min(min(ra, rb));
      // u's root, held by the whole half, and the entries' other roots: one
      // lane hooks each, for all lanes that hold it
      int32_t r = rb != least ? rb : ra;
      bool todo = r != least;
      bool again = false;
      while (__ballot(todo)) {
        const uint64_t m = __ballot(todo);
        const uint32_t mine = half ? (uint32_t)(m >> 32) : (uint32_t)m;
        const int lead = mine ? (half << 5) + __ffs((int)mine) - 1 : lane;
        const int32_t v = __shfl(r, lead, 64);
        int32_t to = v;
        if (todo && lane == lead) {
          to = least;
          if (ld_i32(parent + v) != v || atomicCAS(parent + v, v, least) != v) to = uf_find(parent, v);
        }
        to = __shfl(to, lead, 64);
        if (todo && r == v) {
          todo = false;
          again = to != least;
        }
        if (mine && ra == v) ra = to;
        if (mine && rb == v) rb = to;
      }
      const uint64_t any = __ballot(again || ra != rb || ra != least);
      if (!(half ? (uint32_t)(any >> 32) : (uint32_t)any)) break;
    }
  }
}

__global__ __launch_bounds__(256) void k_tri_attach(int64_t lines, const int32_t* __restrict__ lu,
                                                    const int32_t* __restrict__ oc, const uint32_t* __restrict__ simw,
                                                    const int32_t* __restrict__ lower,
                                                    const int32_t* __restrict__ idof, TriArgs a, int32_t* parent,
                                                    int32_t* label, const int32_t* __restrict__ flag) {
  if (!*flag) return;
  const int sub = threadIdx.x & 31;
  const int64_t stride = (int64_t)gridDim.x * 8;
  for (int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 5; t < lines; t += stride) {
    if (!((simw[t] >> sub) & 1u)) continue;
    const int32_t u = lu[t], x = oc[t * kTriLine + sub] - 1;
    const int32_t mu = tri_mu(a, u);
    const bool cu = lower[u] >= mu, cx = lower[x] >= mu;
    if (cu == cx) continue;
    atomicMin(label + idof[cu ? x : u], uf_find(parent, idof[cu ? u : x]));
  }
}

// Labels of the cores (needed before hub marks, which read every label).
__global__ void k_tri_core_labels(int32_t n, const int32_t* hof, const int32_t* lower, TriArgs a, int32_t* parent,
                                  int32_t* label, int32_t* first) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  if (lower[hof[x]] >= tri_mu(a, x)) label[x] = uf_find(parent, (int32_t)x);
  first[x] = -1;
}

// Def 2.7, one entry per lane: see k_hub_outlier.
__global__ __launch_bounds__(256) void k_tri_hub(int64_t lines, const int32_t* __restrict__ lu,
                                                 const int32_t* __restrict__ oc, const int32_t* __restrict__ idof,
                                                 const int32_t* __restrict__ label, int32_t* first, uint8_t* role,
                                                 const int32_t* __restrict__ flag) {
  if (!*flag) return;
  const int sub = threadIdx.x & 31;
  const int64_t stride = (int64_t)gridDim.x * 8;
  for (int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 5; t < lines; t += stride) {
    const int32_t h = oc[t * kTriLine + sub] - 1;
    if (h < 0) continue;
    const int32_t a = idof[lu[t]], b = idof[h];
    const int32_t la = label[a], lb = label[b];
    if ((la == INT_MAX) == (lb == INT_MAX)) continue;
    const int32_t x = (la == INT_MAX) ? a : b;
    const int32_t L = (la == INT_MAX) ? lb : la;
    const int32_t seen = ld_i32(first + x);
    if (seen == L) continue;
    const int32_t old = (seen == -1) ? atomicCAS(first + x, -1, L) : seen;
    if (old != -1 && old != L) role[x] = ROLE_HUB;
  }
}

__global__ void k_tri_output(int32_t n, const int32_t* __restrict__ hof, const int32_t* __restrict__ lower, TriArgs a,
                             const int64_t* __restrict__ vtx_off, int32_t* parent, const int32_t* __restrict__ label, const uint8_t* __restrict__ role,
                             int32_t* __restrict__ out_labels, uint8_t* __restrict__ out_roles, int32_t split) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const int32_t base = tri_base(a.gid, vtx_off, x);  // labels within the graph
  if (lower[hof[x]] >= tri_mu(a, x)) {
    out_roles[x] = 1;
    out_labels[x] = uf_find(parent, (int32_t)x) - base;
    return;
  }
  const int32_t l = label[x];
  out_labels[x] = l == INT_MAX ? -1 : l - base;
  out_roles[x] = l != INT_MAX ? 2 : split ? (role[x] == ROLE_HUB ? 3 : 4) : 0;
}

// Last row that starts at or before arc i, among rows lo .. hi.
__device__ __forceinline__ int32_t row_of(const int64_t* rp, int32_t lo, int32_t hi, int64_t i) {
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo + 1) / 2;
    if (rp[mid] <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Counts in CSR order; the entry of an arc is found in the row of its endpoint
// with the larger h.  A block takes kTriArcs consecutive arcs, whatever their
// rows (a wave per row left the longest row, some 600 rounds of nine dependent
// loads on R-MAT scale 19, running alone: 2.2 ms; now 0.58 ms).
constexpr int kTriArcs = 1024;
__global__ __launch_bounds__(256) void k_tri_arcs(int32_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                  const int32_t* __restrict__ ci, const int32_t* __restrict__ hof,
                                                  const uint32_t* __restrict__ oline, const int32_t* __restrict__ row,
                                                  const int32_t* __restrict__ oc, const int32_t* __restrict__ cnt,
                                                  int32_t* __restrict__ counts) {
  __shared__ int32_t ends[2];
  const int64_t a0 = (int64_t)blockIdx.x * kTriArcs, a1 = min(a0 + kTriArcs, nnz);
  if ((threadIdx.x & 127) == 0) ends[threadIdx.x >> 7] = row_of(rp, 0, n - 1, threadIdx.x ? a1 - 1 : a0);
  __syncthreads();
  const int32_t r0 = ends[0], r1 = ends[1];
#pragma unroll
  for (int k = 0; k < kTriArcs / 256; ++k) {
    const int64_t i = a0 + k * 256 + threadIdx.x;
    if (i >= a1) continue;
    const int32_t hx = hof[row_of(rp, r0, r1, i)], hy = hof[ci[i]];
    const int32_t u = max(hx, hy), v = min(hx, hy);
    const int64_t base = (int64_t)oline[u] * kTriLine;
    const int32_t j = tri_find(oc + base, row[u], v);
    if (j >= 0) counts[i] = cnt[base + j];
  }
}

inline unsigned grid_for(int64_t items, int64_t per_block) {
  const int64_t b = (items + per_block - 1) / per_block;
  return (unsigned)(b < 1 ? 1 : b);
}

// HIP launches fewer than 2^32 threads at once.
inline bool launchable(int64_t blocks, int64_t threads) { return blocks * threads < (int64_t)1 << 32; }

// Blocks of the counting kernel: its jobs' and its waves' rows'.
int64_t count_blocks(const TriLayout& T) {
  return T.jobs == 0 ? (T.wave_rows + 3) / 4 : T.jobs + (T.wave_rows + kTriBlock / 64 - 1) / (kTriBlock / 64);
}

uint32_t tri_acc_cap(const TriLayout& T) { return ((uint32_t)T.max_row + 2 + 3) & ~3u; }

// Dynamic LDS of the counting kernel: of a job, counters, then the largest table
// of the graph; of waves' rows, a hash set and counters each.
size_t tri_lds_bytes(const TriLayout& T) {
  const size_t rows = 8 * kTriWaveSlots * (kTriBlock / 64);
  const size_t acc = 4 * (size_t)tri_acc_cap(T);
  size_t b = acc + 2 * ((size_t)std::min(T.span, kTriDirect) + 24);
  if (T.span > kTriDirect) b = std::max(b, acc + 8 * ((size_t)std::min(T.span, kTriShort) / 32 + 3));
  if (T.max_hash_row > 0) b = std::max(b, 8 * (size_t)tri_hash_slots(T.max_hash_row));
  return std::max((b + 15) & ~(size_t)15, rows);
}

// Several arrays in one allocation (allocating and freeing some thirty of them
// took longer than the kernels that build the layout): take() them, allocate, and
// their pointers are set.
class Arena {
 public:
  template <typename T>
  void take(T** p, int64_t count) {
    slots_.push_back({reinterpret_cast<void**>(p), total_});
    total_ += (sizeof(T) * (size_t)(count > 0 ? count : 1) + 255) & ~(size_t)255;
  }
  hipError_t allocate(void** mem) {
    const hipError_t e = hipMalloc(mem, total_);
    if (e != hipSuccess) {
      *mem = nullptr;
      return e;
    }
    for (const auto& s : slots_) *s.first = static_cast<char*>(*mem) + s.second;
    return hipSuccess;
  }

 private:
  std::vector<std::pair<void**, size_t>> slots_;
  size_t total_ = 0;
};

}  // namespace

namespace {

uint64_t row_bytes(const TriLayout& T) {  // per vertex and per line
  const uint64_t n = (uint64_t)T.n, L = (uint64_t)T.lines;
  return 16 * n + 8 * (n + 1) + 20 * L + 4 * (L + 2) * kTriLine;
}

uint64_t input_bytes(const TriLayout& T) {  // what tri_drop_inputs frees
  return 2 * ((uint64_t)T.lines + 2) * kTriLine + sizeof(TriRec) * (uint64_t)T.recs + sizeof(TriJob) * (uint64_t)T.jobs +
         sizeof(TriWave) * (uint64_t)T.wave_rows;
}

// A layout of T's sizes and its scratches.
uint64_t tri_bytes(const TriLayout& T, int scratches) {
  const uint64_t L = (uint64_t)T.lines;
  return row_bytes(T) + input_bytes(T) + (uint64_t)scratches * (4 * L * kTriLine + 4 * (uint64_t)T.words + 4 * L + 4);
}

}  // namespace

uint64_t tri_layout_bytes(const TriLayout& T) { return row_bytes(T) + (T.oc16 ? input_bytes(T) : 0); }

uint64_t tri_scratch_bytes(const TriLayout& T, const TriScratch& S) {
  const uint64_t L = (uint64_t)T.lines;
  return (S.cnt ? 4 * L * kTriLine : 0) + (S.bits ? 4 * (uint64_t)T.words : 0) + (S.simw ? 4 * L : 0) + (S.flag ? 4 : 0);
}

void tri_drop_inputs(TriLayout& T) {
  for (int k = 2; k < 4; ++k) {
    if (T.mem[k]) (void)hipFree(T.mem[k]);
    T.mem[k] = nullptr;
  }
  T.oc16 = nullptr;
  T.rec = nullptr;
  T.job = nullptr;
  T.wrow = nullptr;
}

void tri_release(TriLayout& T) {
  for (void* m : T.mem)
    if (m) (void)hipFree(m);
  T = TriLayout();
}

void tri_drop_work(TriScratch& S) {
  if (S.mem) (void)hipFree(S.mem);
  S.mem = nullptr;
  S.bits = nullptr;
  S.simw = nullptr;
  S.flag = nullptr;
}

void tri_release_scratch(TriScratch& S) {
  tri_drop_work(S);
  if (S.cnt) (void)hipFree(S.cnt);
  S = TriScratch();
}

uint64_t tri_place_scratch(const TriLayout& T, unsigned char* base, TriScratch* S) {
  // (no container here: a no-alloc call must not allocate on the host either)
  const uint64_t bytes[4] = {4 * (uint64_t)T.lines * kTriLine, 4 * (uint64_t)T.words, 4 * (uint64_t)T.lines, 4};
  uint64_t at[5] = {0};
  for (int k = 0; k < 4; ++k) at[k + 1] = at[k] + ((bytes[k] + 255) & ~255ull);
  if (S) {
    *S = TriScratch();
    S->cnt = reinterpret_cast<int32_t*>(base);
    S->bits = reinterpret_cast<uint32_t*>(base + at[1]);
    S->simw = reinterpret_cast<uint32_t*>(base + at[2]);
    S->flag = reinterpret_cast<int32_t*>(base + at[3]);
  }
  return at[4];
}

hipError_t tri_alloc_scratch(const TriLayout& T, TriScratch* S) {
  Arena work;
  work.take(&S->bits, T.words);
  work.take(&S->simw, T.lines);
  work.take(&S->flag, 1);
  hipError_t e = work.allocate(&S->mem);
  if (e == hipSuccess) e = hipMalloc((void**)&S->cnt, 4 * (size_t)std::max<int64_t>(T.lines * kTriLine, 1));
  if (e != hipSuccess) {
    S->cnt = nullptr;
    tri_release_scratch(*S);
  }
  return e;
}

hipError_t tri_build(hipStream_t s, int32_t n, int64_t nnz, const int64_t* h_rp, const int64_t* d_rp,
                     const int32_t* d_ci, const LayoutResult& csr, const TriGroups* groups, int scratches,
                     uint64_t max_bytes, TriLayout* out, int64_t* bucket_edges, int* ok) {
  *ok = 0;
  if (n <= 0 || nnz <= 0 || nnz / 2 >= (int64_t)1 << 31) return hipSuccess;
  // The kernels below take a wave per vertex: up to 67,108,860 vertices (more than
  // that seldom fit the limit on lines either, one per vertex and up).
  if (!launchable(grid_for(n, 4), 256)) return hipSuccess;
  TriLayout T;
  T.n = n;
  hipError_t e = hipSuccess;
  int64_t *nline = nullptr, *nword = nullptr, *nin = nullptr, *at0 = nullptr, *at1 = nullptr, *at2 = nullptr;
  int64_t* work = nullptr;
  // Records per wave of the wave kernel.  A wave goes through its records one
  // after the other (512 of them: 120 us, all of a small graph's time), but builds
  // its row's table first.  Kernel, in parts of up to 512, 128, 64 and 32 records:
  // R-MAT scale 14 (m = 0.2 M) 120, 53, 30, 18 us; scale 17 (1.9 M) 54, 54, 43, 37;
  // scale 19 (5.9 M) 258, 173, 150, 156; scale 22 (64 M) 490, 490, 496, 526; Chung-Lu
  // (7.4 M) 250, 217, 220, 229.  300 planted graphs (20 M) 773, 773, 792, 867.
  const uint32_t part = nnz / 2 < (4 << 20) ? 32 : nnz / 2 < (16 << 20) ? 64 : 128;
  uint32_t* inlen = nullptr;
  uint8_t* wcls = nullptr;
  void* tmp = nullptr;
  int32_t *ctl = nullptr, *longer = nullptr;
  BigChunk* big = nullptr;
  std::vector<BigChunk> chunks;
  unsigned long long* room = nullptr;
  unsigned nchunk = 0;
  unsigned long long* sums = nullptr;
  int64_t tot[4] = {0, 0, 0, 0};
  int32_t h_ctl[4] = {0, 0, 0, 0};
  unsigned long long h_sums[2 + kNumBuckets] = {0};
  const unsigned gv = grid_for((int64_t)n + 1, 256);
  const int32_t nbig = groups ? 0 : csr.long_rows;  // (of a batch, waves take the long rows too)
  // vertices from here on have few neighbours, and go eight to a wave
  const int32_t narrow = !groups && n - csr.wide_rows >= kNarrowWorth ? csr.wide_rows : n;
  int32_t few = n;  // vertices from here on are left to k_tri_few
  int64_t* digits = nullptr;
#define TTRY(x)                        \
  do {                                 \
    e = (x);                           \
    if (e != hipSuccess) goto done;    \
  } while (0)
  T.span = n;
  if (groups) {
    T.vtx_off = groups->vtx_off;
    T.gid = groups->gid;
    T.span = 0;
    for (int32_t k = 0; k < groups->count; ++k)
      T.span = std::max(T.span, (int32_t)(groups->h_vtx_off[k + 1] - groups->h_vtx_off[k]));
  }
  {
    Arena vertex, temp;
    vertex.take(&T.hof, n);
    vertex.take(&T.idof, n);
    vertex.take(&T.deg, n);
    vertex.take(&T.row, n);
    vertex.take(&T.oline, (int64_t)n + 1);
    vertex.take(&T.wbase, (int64_t)n + 1);
    TTRY(vertex.allocate(&T.mem[0]));
    for (int64_t** p : {&nline, &nword, &nin, &at0, &at1, &at2}) temp.take(p, (int64_t)n + 1);
    temp.take(&digits, 2 * sort_counts(n));
    temp.take(&work, scan_work_items(std::max((int64_t)n + 1, sort_counts(n))));
    temp.take(&inlen, n);
    temp.take(&wcls, n);
    temp.take(&longer, n);
    temp.take(&ctl, 4);  // longest row, rows for the block sort, longest hash row, a reverse arc is missing
    temp.take(&sums, 2 + kNumBuckets);  // words, edges per bucket, entries
    temp.take(&big, nbig + nnz / kTriBigChunk);
    temp.take(&room, 2 * (int64_t)nbig);
    TTRY(temp.allocate(&tmp));
  }
  if (groups) {
    std::vector<int32_t> hof((size_t)n);
    rename_groups(h_rp, *groups, hof.data());
    TTRY(hipMemcpyAsync(T.hof, hof.data(), 4 * (size_t)n, hipMemcpyHostToDevice, s));
    k_inverse<<<gv, 256, 0, s>>>(n, T.hof, T.idof);
    TTRY(hipGetLastError());
    TTRY(hipStreamSynchronize(s));
  } else {
    TTRY(sort_by_degree(s, n, d_rp, csr.max_degree, reinterpret_cast<int2*>(nline), reinterpret_cast<int2*>(nword),
                        digits, work, T.hof, T.idof));
  }
  if (nbig > 0) {
    std::vector<int32_t> ids((size_t)nbig);
    TTRY(hipMemcpyAsync(ids.data(), T.idof, 4 * (size_t)nbig, hipMemcpyDeviceToHost, s));
    TTRY(hipStreamSynchronize(s));
    for (int32_t h = 0; h < nbig; ++h) {
      const int32_t v = ids[(size_t)h];
      for (int64_t k = h_rp[v]; k < h_rp[v + 1]; k += kTriBigChunk)
        chunks.push_back(BigChunk{h, v, k, std::min(k + kTriBigChunk, h_rp[v + 1])});
    }
    nchunk = (unsigned)chunks.size();
    TTRY(hipMemcpyAsync(big, chunks.data(), sizeof(BigChunk) * nchunk, hipMemcpyHostToDevice, s));
    TTRY(hipMemsetAsync(room, 0, 16 * (size_t)nbig, s));
  }
  TTRY(hipMemsetAsync(ctl, 0, 16, s));
  TTRY(hipMemsetAsync(sums, 0, sizeof(h_sums), s));
  k_degrees<<<gv, 256, 0, s>>>(n, d_rp, T.idof, T.deg, T.row);
  if (nchunk) k_row_len_block<<<nchunk, 256, 0, s>>>(big, d_ci, T.hof, T.row);
  if (narrow > nbig)
    k_row_len_wave<64><<<grid_for(narrow - nbig, 4), 256, 0, s>>>(nbig, narrow, d_rp, d_ci, T.hof, T.idof, T.row);
  if (n > narrow)
    k_row_len_wave<8><<<grid_for(n - narrow, 32), 256, 0, s>>>(narrow, n, d_rp, d_ci, T.hof, T.idof, T.row);
  TTRY(hipGetLastError());
  k_row_sizes<<<std::min(gv, 512u), 256, 0, s>>>(n, T.row, nline, nword, sums + 1 + kNumBuckets, ctl);
  if (nchunk) {
    k_in_room_block<<<nchunk, 256, 0, s>>>(big, d_ci, T.hof, T.row, room);
    k_in_room_big<<<grid_for(nbig, 256), 256, 0, s>>>(nbig, T.row, room, nin, wcls);
  }
  if (narrow > nbig)
    k_in_room_wave<64><<<grid_for(narrow - nbig, 4), 256, 0, s>>>(nbig, narrow, d_rp, d_ci, T.hof, T.idof, T.row, nin,
                                                                  wcls);
  if (n > narrow)
    k_in_room_wave<8><<<grid_for(n - narrow, 32), 256, 0, s>>>(narrow, n, d_rp, d_ci, T.hof, T.idof, T.row, nin, wcls);
  TTRY(hipMemsetAsync(nin + n, 0, 8, s));
  TTRY(hipGetLastError());
  TTRY(exclusive_scan(s, nline, at0, (int64_t)n + 1, work));
  TTRY(exclusive_scan(s, nword, at1, (int64_t)n + 1, work));
  TTRY(exclusive_scan(s, nin, at2, (int64_t)n + 1, work));
  TTRY(hipMemcpyAsync(tot + 0, at0 + n, 8, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(tot + 1, at1 + n, 8, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(tot + 2, at2 + n, 8, hipMemcpyDeviceToHost, s));
  if (narrow < n) TTRY(hipMemcpyAsync(tot + 3, at2 + narrow, 8, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(h_ctl, ctl, 16, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(h_sums, sums, sizeof(h_sums), hipMemcpyDeviceToHost, s));
  TTRY(hipStreamSynchronize(s));
  T.max_row = h_ctl[0];
  T.lines = tot[0];
  T.words = tot[1];
  T.recs = tot[2];
  // Where most records are those of vertices of few neighbours, k_tri_few takes
  // them.  (Elsewhere they stay with the waves: taken out of R-MAT scale 22, where
  // they are few and k_tri_few needs 10 us, the blocks left in k_tri_count went from
  // 6.9 to 8.1 ms.)
  few = narrow < n && T.recs - tot[3] >= T.recs / 2 ? narrow : n;
  T.few_at = few < n ? tot[3] : T.recs;
  T.few = T.recs - T.few_at;
  // outside the limits (32-bit byte offsets of 16-bit entries and of bits), or not a symmetric CSR
  if (T.max_row > kTriMaxRow || T.lines >= (int64_t)1 << 26 || T.words >= (int64_t)1 << 30 ||
      T.recs >= (int64_t)1 << 32 || (int64_t)h_sums[1 + kNumBuckets] != nnz / 2)
    goto done;
  if (tri_bytes(T, scratches) > max_bytes) goto done;
  k_narrow<<<gv, 256, 0, s>>>(n, at0, at1, T.oline, T.wbase);
  {
    Arena rows, inputs;
    rows.take(&T.lu, T.lines);
    rows.take(&T.li, T.lines);
    // steps of 64 entries may start on a row's last line
    rows.take(&T.oc, (T.lines + 2) * kTriLine);
    TTRY(rows.allocate(&T.mem[1]));
    inputs.take(&T.oc16, (T.lines + 2) * kTriLine);
    inputs.take(&T.rec, T.recs);
    TTRY(inputs.allocate(&T.mem[2]));
  }
  TTRY(hipMemsetAsync(inlen, 0, 4 * (size_t)n, s));  // here: entries of the big rows so far
  if (nchunk) {
    k_row_fill_block<<<nchunk, 256, 0, s>>>(big, d_ci, T.hof, T.oline, T.row, inlen, T.oc);
    k_row_pad<<<grid_for(nbig, 8), 256, 0, s>>>(nbig, T.oline, T.row, T.oc);
  }
  if (narrow > nbig)
    k_row_fill_wave<64><<<grid_for(narrow - nbig, 4), 256, 0, s>>>(nbig, narrow, d_rp, d_ci, T.hof, T.idof, T.oline,
                                                                   T.row, T.oc);
  if (n > narrow)
    k_row_fill_wave<8><<<grid_for(n - narrow, 32), 256, 0, s>>>(narrow, n, d_rp, d_ci, T.hof, T.idof, T.oline, T.row,
                                                                T.oc);
  if (narrow > 0)
    k_row_sort_wave<64><<<grid_for(narrow, 4), 256, 0, s>>>(0, narrow, T.oline, T.row, T.wbase, T.deg, T.gid, T.vtx_off,
                                                            T.oc, T.oc16, T.lu, T.li, longer, ctl + 1);
  if (n > narrow)
    k_row_sort_wave<8><<<grid_for(n - narrow, 32), 256, 0, s>>>(narrow, n, T.oline, T.row, T.wbase, T.deg, T.gid,
                                                                T.vtx_off, T.oc, T.oc16, T.lu, T.li, longer, ctl + 1);
  k_row_sort_block<<<4096, 256, 0, s>>>(longer, ctl + 1, T.oline, T.row, T.gid, T.vtx_off, T.oc, T.oc16);
  TTRY(hipGetLastError());
  TTRY(hipMemsetAsync(inlen, 0, 4 * (size_t)n, s));
  TTRY(hipMemsetAsync(nin, 0, 8 * (size_t)n, s));  // from here on: words of every vertex's in-edges
  if (nchunk)
    k_recs_block<<<nchunk, 256, 0, s>>>(big, d_ci, T.hof, T.oline, T.wbase, T.row, T.oc, at2, wcls, T.rec, inlen, nin,
                                        ctl + 3);
  if (narrow > nbig)
    k_recs_wave<64><<<grid_for(narrow - nbig, 4), 256, 0, s>>>(nbig, narrow, d_rp, d_ci, T.hof, T.idof, T.oline, T.wbase,
                                                               T.row, T.oc, at2, wcls, T.rec, inlen, nin, ctl + 3);
  if (n > narrow)
    k_recs_wave<8><<<grid_for(n - narrow, 32), 256, 0, s>>>(narrow, n, d_rp, d_ci, T.hof, T.idof, T.oline, T.wbase,
                                                            T.row, T.oc, at2, wcls, T.rec, inlen, nin, ctl + 3);
  k_job_counts<<<std::min(gv, 512u), 256, 0, s>>>(n, few, T.gid, T.vtx_off, T.row, wcls, inlen, nin, nline, nword, part, sums,
                                                ctl + 2);
  k_tri_buckets<<<grid_for(std::min<int64_t>(T.lines * kTriLine, 1 << 22), 1024), 256, 0, s>>>(T.lines, T.lu, T.oc,
                                                                                               T.deg, sums + 1);
  TTRY(hipGetLastError());
  TTRY(exclusive_scan(s, nline, at0, (int64_t)n + 1, work));
  TTRY(exclusive_scan(s, nword, at1, (int64_t)n + 1, work));
  TTRY(hipMemcpyAsync(tot + 0, at0 + n, 8, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(tot + 1, at1 + n, 8, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(h_ctl, ctl, 16, hipMemcpyDeviceToHost, s));
  TTRY(hipMemcpyAsync(h_sums, sums, sizeof(h_sums), hipMemcpyDeviceToHost, s));
  TTRY(hipStreamSynchronize(s));
  if (h_ctl[3]) goto done;  // not a symmetric CSR
  T.jobs = tot[0];
  T.wave_rows = tot[1];
  T.max_hash_row = h_ctl[2];
  T.steps = (int64_t)h_sums[0];
  if (tri_bytes(T, scratches) > max_bytes) goto done;  // with the jobs
  if (!launchable(count_blocks(T), T.jobs == 0 ? 256 : kTriBlock)) goto done;
  for (int k = 0; k < kNumBuckets; ++k) bucket_edges[k] = (int64_t)h_sums[1 + k];
  {
    Arena jobs;
    jobs.take(&T.job, T.jobs);
    jobs.take(&T.wrow, T.wave_rows);
    TTRY(jobs.allocate(&T.mem[3]));
  }
  k_job_fill<<<gv, 256, 0, s>>>(n, at2, inlen, T.oline, T.row, at0, at1, part, T.job, T.wrow);
  TTRY(hipGetLastError());
  TTRY(hipStreamSynchronize(s));
  *out = T;
  *ok = 1;
done:
  (void)hipStreamSynchronize(s);
  if (tmp) (void)hipFree(tmp);
  if (!*ok) tri_release(T);
#undef TTRY
  return e;
}

void tri_init(hipStream_t s, const TriLayout& T, const TriScratch& S, int32_t* lower, int32_t* parent,
              int32_t* label, uint8_t* role) {
  const int64_t ncnt4 = T.lines * (kTriLine / 4);
  const unsigned grid = (unsigned)std::min<int64_t>(grid_for(std::max<int64_t>(ncnt4, T.n), 256), 8192);
  k_tri_init<<<grid, 256, 0, s>>>(ncnt4, reinterpret_cast<int4*>(S.cnt), T.n, lower, parent, label, role, S.flag);
}

void tri_init_state(hipStream_t s, const TriLayout& T, const TriScratch& S, int32_t* lower, int32_t* parent,
                    int32_t* label, uint8_t* role) {
  const unsigned grid = (unsigned)std::min<int64_t>(grid_for(T.n, 256), 8192);
  k_tri_init<<<grid, 256, 0, s>>>(0, nullptr, T.n, lower, parent, label, role, S.flag);
}

void tri_threshold(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, int32_t* lower) {
  if (T.lines > 0)
    k_tri_threshold<<<grid_for(T.lines, 8), 256, 0, s>>>(T.lines, T.li, T.deg, T.oc, S.cnt, a, S.simw, lower);
}

void tri_count(hipStream_t s, const TriLayout& T, const TriScratch& S) {
  if (T.few > 0)
    k_tri_few<<<grid_for(T.few, 256), 256, 0, s>>>(T.few, T.rec + T.few_at, T.row, T.oline, T.oc, S.bits, S.cnt);
  if (T.jobs == 0) {
    if (T.wave_rows == 0) return;
    const unsigned grid = (unsigned)count_blocks(T);
    if (T.span <= kTriShort)
      k_tri_wave<<<grid, 256, 0, s>>>(T.wave_rows, T.wrow, T.rec, T.oc16, T.lines, S.bits, S.cnt);
    else
      k_tri_wave<<<grid, 256, 0, s>>>(T.wave_rows, T.wrow, T.rec, reinterpret_cast<const uint32_t*>(T.oc), T.lines,
                                      S.bits, S.cnt);
    return;
  }
  const uint64_t blocks = (uint64_t)count_blocks(T);
  // rounded up: exactly T.jobs of the products blocks * ratio step over a whole number
  const uint64_t ratio = (((uint64_t)T.jobs << 32) + blocks - 1) / blocks;
  const auto launch = T.span <= kTriShort ? k_tri_count<uint16_t> : k_tri_count<uint32_t>;
  launch<<<(unsigned)blocks, kTriBlock, tri_lds_bytes(T), s>>>(ratio, T.job, T.wave_rows, T.wrow, T.rec, T.row, T.oline,
                                                               T.gid, T.vtx_off, T.oc, T.oc16, T.lines, S.bits, S.cnt,
                                                               tri_acc_cap(T));
}

void tri_close(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, int32_t* lower) {
  if (T.lines <= 0) return;
  const unsigned grid = grid_for(T.lines, 8);
  if (a.q || a.gq)
    k_tri_close<true><<<grid, 256, 0, s>>>(T.lines, T.li, T.deg, T.oc, S.bits, S.cnt, a, S.simw, lower);
  else
    k_tri_close<false><<<grid, 256, 0, s>>>(T.lines, T.li, T.deg, T.oc, S.bits, S.cnt, a, S.simw, nullptr);
}

namespace {
unsigned line_grid(const TriLayout& T) { return (unsigned)std::min<int64_t>(grid_for(T.lines, 8), 1 << 16); }
}  // namespace

void tri_hook(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, const int32_t* lower,
              int32_t* parent) {
  if (T.lines <= 0) return;
  k_tri_link<<<line_grid(T), 256, 0, s>>>(T.lines, T.lu, T.oc, S.simw, lower, T.idof, a, parent, S.flag);
  k_tri_compress<<<grid_for(T.n, 256), 256, 0, s>>>(T.n, parent, S.flag);
  k_tri_hook<<<line_grid(T), 256, 0, s>>>(T.lines, T.lu, T.oc, S.simw, lower, T.idof, a, parent, S.flag);
}

void tri_attach(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, const int32_t* lower,
                int32_t* parent, int32_t* label) {
  if (T.lines > 0)
    k_tri_attach<<<line_grid(T), 256, 0, s>>>(T.lines, T.lu, T.oc, S.simw, lower, T.idof, a, parent, label, S.flag);
}

void tri_hub_outlier(hipStream_t s, const TriLayout& T, const TriScratch& S, const TriArgs& a, const int32_t* lower,
                     int32_t* parent, int32_t* label, int32_t* first, uint8_t* role) {
  k_tri_core_labels<<<grid_for(T.n, 256), 256, 0, s>>>(T.n, T.hof, lower, a, parent, label, first);
  if (T.lines > 0)
    k_tri_hub<<<line_grid(T), 256, 0, s>>>(T.lines, T.lu, T.oc, T.idof, label, first, role, S.flag);
}

void tri_output(hipStream_t s, const TriLayout& T, const TriArgs& a, const int32_t* lower, int32_t* parent,
                const int32_t* label, const uint8_t* role, int32_t* out_labels, uint8_t* out_roles, int32_t split) {
  if (T.n > 0)
    k_tri_output<<<grid_for(T.n, 256), 256, 0, s>>>(T.n, T.hof, lower, a, T.vtx_off, parent, label, role, out_labels,
                                                    out_roles, split);
}

void tri_arc_counts(hipStream_t s, const TriLayout& T, const TriScratch& S, int64_t nnz, const int64_t* rp,
                    const int32_t* ci, int32_t* counts) {
  if (nnz > 0)
    k_tri_arcs<<<grid_for(nnz, kTriArcs), 256, 0, s>>>(T.n, nnz, rp, ci, T.hof, T.oline, T.row, T.oc, S.cnt, counts);
}

}  // namespace scan
