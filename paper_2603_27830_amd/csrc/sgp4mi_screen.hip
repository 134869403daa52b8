// Conjunction screening on the propagation output: every pair of satellites
// closer than a distance D at a common sample time.
//
// The paper motivates batched propagation by catalogue-wide tasks such as
// conjunction screening (sections 1 and 6) without defining one; this is the
// screening step as defined in the header: at each sample time k, every pair
// i < j of points whose states are valid with
//     d2 = (dx*dx + dy*dy) + dz*dz < D*D,
// dx = x_j - x_i (and so on) formed in double from the stored positions, is an
// event (i, j, k, sqrt(d2)).
//
// Two paths.  The usual one (mode 0 and 1): a packing pass writes the float x,
// y and z of every valid point time-major into the workspace (64 x 64 tiles
// through LDS, so that both the reads along times and the writes along
// satellites are coalesced; invalid points get x = +inf), and the largest
// |x| or |y| and the largest |z| of each slot of times.  A second pass counts
// each time's points by strips of x, deals the strips out as sets of equally many
// points, and writes a class byte per point that names its set.  Then workgroups
// of 1,024 lanes each take one sample time and one set of it: they stream the
// time's class bytes, collect the points of their set in LDS in a hash table of
// (x, y) cells, and test each point against the cells that can hold a partner.
// The other path (mode 2, and catalogues beyond kSlabMaxN) sorts buckets of x in
// device memory.
//
// A candidate is taken to the exact test, on the stored positions, when its
// float coordinates are within D plus a rounding margin in every axis.  The
// margin, 2.4e-7 R for coordinates up to R (one R for x and y, one for z), covers
// the two roundings (2^-24 relative each), so no pair closer than D is pruned.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

namespace sgp4mi {

constexpr int kScreenMaxN = 12288;  // largest n of mode 1

template <class TR>
__device__ __forceinline__ double dist2(const TR* __restrict__ r, int64_t P, int64_t pi, int64_t pj) {
#pragma clang fp contract(off)
  const double dx = double(r[pj]) - double(r[pi]);
  const double dy = double(r[P + pj]) - double(r[P + pi]);
  const double dz = double(r[2 * P + pj]) - double(r[2 * P + pi]);
  return (dx * dx + dy * dy) + dz * dz;
}

// ---------------------------------------------------------- column path --
// Workspace: a slot per sixteen time tiles, a class byte per point (rows of T,
// each padded to whole words), then x, y and z as [T][n] floats.
constexpr int kSlots = 16;
// What the sample times of one slot (time tiles of 64 in turn) share: the bits of
// the largest |x| or |y| and of the largest |z| (non-negative floats order as
// integers), and the height of the rows in column widths.
struct SlabSlot {
  uint32_t rxy, rz;
  uint32_t rows;  // float bits
  uint32_t pad;
};
static_assert(kSlots * sizeof(SlabSlot) == 256, "the workspace's first 256 bytes");

constexpr float kRowsMax = 16.0f;

struct SlabLayout {
  SlabSlot* slots;
  uint32_t* cls;  // [T][words]
  float *x, *y, *z;
  int64_t words;
};

__device__ __forceinline__ int slot_of(int64_t k) { return int((k >> 6) & (kSlots - 1)); }

static SlabLayout slab_layout(void* ws, int64_t n, int64_t T) {
  SlabLayout L;
  L.words = (n + 3) / 4;
  L.slots = static_cast<SlabSlot*>(ws);
  L.cls = reinterpret_cast<uint32_t*>(L.slots + kSlots);
  L.x = reinterpret_cast<float*>(L.cls + L.words * T);
  L.y = L.x + n * T;
  L.z = L.y + n * T;
  return L;
}

// 13 bytes a point and a little: within the device-memory path's workspace.
static size_t slab_ws_bytes(int64_t n, int64_t T) {
  return sizeof(SlabSlot) * kSlots + 4 * (size_t((n + 3) / 4) * size_t(T) + 3 * size_t(n) * size_t(T));
}

__global__ void __launch_bounds__(64) slab_clear(SlabLayout L, unsigned long long* count) {
  if (threadIdx.x == 0) *count = 0ull;
  if (threadIdx.x < kSlots) L.slots[threadIdx.x] = SlabSlot{0u, 0u, __float_as_uint(kRowsMax), 0u};
}

// Cells of a slot's times.  near, near_z: the float distance along x or y, and
// along z, of any pair closer than D; reach: the column width, which also covers
// the roundings of a coordinate times its reciprocal (2^-24 of up to R / w each).
struct Cells {
  float near, near_z, reach, inv_w;
};
__device__ __forceinline__ Cells cells_of(const SlabSlot& s, double D) {
  const double R = double(__uint_as_float(s.rxy)), Rz = double(__uint_as_float(s.rz));
  Cells c;
  c.near = float((D + 2.4e-7 * R) * (1.0 + 1.0e-6));
  c.near_z = float((D + 2.4e-7 * Rz) * (1.0 + 1.0e-6));
  c.reach = float((D + 8.0e-7 * R) * (1.0 + 1.0e-5));
  c.inv_w = 1.0f / c.reach;
  return c;
}

// Rows (cells along y) are this many column widths tall, for n points spread over
// a sphere of l columns radius.  A point looks up its own cell, the one above when
// it is within reach, and one or two of the next column: tall rows mean fewer
// lookups, but a cell should rarely hold a point (it holds about 0.6 n h / l^2 on
// average; the factor aims at 0.15).  Below two widths a point could reach both
// neighbours.
__device__ __forceinline__ float row_widths(float l, float n) {
  return fminf(fmaxf(0.25f * l * l / n, 2.5f), kRowsMax);
}

// Column of x: below 1.3 million in size for every valid point.
__device__ __forceinline__ int32_t column_of(float x, float inv_w) { return int32_t(floorf(x * inv_w)); }

// A finite double beyond float's range as float's largest (its points only meet
// each other, and the exact test decides on the stored positions).
__device__ __forceinline__ float in_float(float z) { return z; }
__device__ __forceinline__ float in_float(double z) { return float(fmin(fmax(z, -3.4028234663852886e38), 3.4028234663852886e38)); }

// Pack one 64 x 64 tile.  A lane has its 48 position loads (16 points) out
// before it uses one: 9,341 x 1,000 floats 54 us for three coordinates, against
// 60 for two when each point's loads were waited for in turn.
template <class TR>
__global__ void __launch_bounds__(256) screen_pack(const TR* __restrict__ r, const uint8_t* __restrict__ err, int64_t n,
                                                   int64_t T, SlabLayout L) {
  __shared__ float tile[64][65];
  __shared__ float wave_max[2][4];
  const int64_t k0 = int64_t(blockIdx.x) * 64, i0 = int64_t(blockIdx.y) * 64;  // times on x: T may be large
  const int64_t P = n * T;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  TR c[3][16];
  uint8_t code[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {  // consecutive lanes: consecutive times of one satellite
    const int64_t i = i0 + wave + 4 * q, k = k0 + lane;
    const bool in = i < n && k < T;
    const int64_t p = in ? i * T + k : 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) c[d][q] = in ? r[d * P + p] : TR(0);
    code[q] = in && err ? err[p] : uint8_t(0);
  }
  float most = 0.0f, most_z = 0.0f;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const float x = float(c[0][q]), y = float(c[1][q]), z = in_float(c[2][q]);
    const bool ok = isfinite(x) && isfinite(y) && isfinite(double(c[2][q])) && (code[q] == 0 || code[q] == 6);
    if (ok) {
      most = fmaxf(most, fmaxf(fabsf(x), fabsf(y)));
      most_z = fmaxf(most_z, fabsf(z));
    } else {
      c[0][q] = TR(__builtin_inff());
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    most = fmaxf(most, __shfl_xor(most, o));
    most_z = fmaxf(most_z, __shfl_xor(most_z, o));
  }
  if (lane == 0) {
    wave_max[0][wave] = most;
    wave_max[1][wave] = most_z;
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    float* const out = d == 0 ? L.x : d == 1 ? L.y : L.z;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) tile[wave + 4 * q][lane] = d == 2 ? in_float(c[d][q]) : float(c[d][q]);
    __syncthreads();
    const int64_t i = i0 + lane;  // consecutive lanes: consecutive satellites at one time
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int64_t k = k0 + wave + 4 * q;
      if (i < n && k < T) out[k * n + i] = tile[lane][wave + 4 * q];
    }
  }
  if (threadIdx.x < 2) {
    const float* const m = wave_max[threadIdx.x];
    SlabSlot& slot = L.slots[slot_of(k0)];
    atomicMax(threadIdx.x == 0 ? &slot.rxy : &slot.rz, __float_as_uint(fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]))));
  }
}

// Strips of columns, in their order, fine near the origin and 1/256 of the distance
// from it beyond 64 columns: whatever the range of x, a strip of the densest part
// holds a small share of the points.  With v = 64 + the column's distance from the
// origin, a strip is the leading eight bits of v's fraction at v's exponent: 256
// strips per doubling, 15 doublings to the largest column.  Columns are taken as
// floats here (exact below 2^23).
constexpr int kStripShift = 23 - 8, kStrips = 8192;
constexpr uint32_t kStripZero = 0x42800000u >> kStripShift;  // 64.0f
__device__ __forceinline__ uint32_t strip_of(float column) {
  const float v = fminf(fabsf(column + 0.5f) + 63.5f, 0x1p21f);
  const uint32_t s = __float_as_uint(v) >> kStripShift;
  return column < 0.0f ? kStrips / 2 - 1 + kStripZero - s : kStrips / 2 - kStripZero + s;
}
// The first column of a strip that has one.
__device__ __forceinline__ float strip_column(uint32_t strip) {
  const uint32_t half = kStrips / 2;
  if (strip >= half) return ceilf(__uint_as_float((strip - half + kStripZero) << kStripShift)) - 64.0f;
  return 64.0f - ceilf(__uint_as_float((half - strip + kStripZero) << kStripShift));
}
// Columns of a strip (the strips of the first two doublings are finer than a column).
__device__ __forceinline__ float strip_columns(uint32_t strip) {
  const uint32_t s = strip < kStrips / 2 ? kStrips / 2 - 1 - strip : strip - kStrips / 2;
  return s < 3u << 8 ? 1.0f : float(1 << ((s >> 8) - 2));
}

// Class byte of every point: its column set and, in bit 7, whether its column is
// the first of a run; invalid points 0xff.  The column sets' workgroups then test
// four points per instruction.
//
// Runs of strips share a time's points evenly, so they follow the points and not
// the largest coordinate (blocks of equal width over [-R, R] put 3,817 of 9,341 low
// satellites into one of five sets when another one is at 42,164 km, and 9,340
// when it is at 120,000 km).  A set is two runs half the range apart, since cells
// near the limb hold more points than those at the centre; where a column holds
// more than kTwoRunsColumn points, whose copies above each run would crowd the
// table, it is one.  A workgroup counts its time's points by strip in LDS (beyond
// 16,384 satellites one of each of so many stretches of them: a run's share comes
// out within a tenth or so), numbers the strips' runs, and writes its part of the
// class bytes.  A run begins at the strip that holds a multiple of the share in
// its first half, or after the one that holds it in its second; only strips with
// counted points begin one, so that the runs are numbered in the order of x
// without gaps and the points next to a run's upper edge are the first column of
// the next number.  The mean density around a point gives the rows' height.
//
// Bound by latency (a load, the counts, two sums over the workgroup) and, over many
// times, by VALU issue: all loads are out before one is used.  9,341 x 100 13 us,
// 100,000 x 144 43 us; the class bytes from equal blocks and their geometry took 8
// and 27, the sweep then 21 and 523 instead of 18 and 479.
constexpr int kSetsBlock = 1024, kSetsWaves = kSetsBlock / 64;
constexpr int kSetSamples = 1 << 14;
constexpr float kTwoRunsColumn = 200.0f;
__global__ void __launch_bounds__(kSetsBlock)
    screen_sets(SlabLayout L, int32_t n, int64_t T, double D, int32_t slabs, int32_t parts, int32_t part_words) {
  constexpr int kOwn = kStrips / kSetsBlock, kLoads = kSetSamples / kSetsBlock;
  static_assert(kOwn == 8 && kSetsWaves == 16, "two loads of four counts, one store of eight numbers; sums of sixteen");
  __shared__ __align__(16) int4 count[kStrips / 4];
  __shared__ uint64_t run_of[kStrips / 8];
  __shared__ float run_column[256];  // a run's first column
  __shared__ int32_t wave_points[kSetsWaves], wave_last[kSetsWaves], wave_begins[kSetsWaves];
  __shared__ float wave_dense[kSetsWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t k = blockIdx.x / parts;
  const int32_t word0 = int32_t(blockIdx.x - k * parts) * part_words, words = int32_t(L.words);
  const int32_t word1 = word0 + part_words < words ? word0 + part_words : words;
  const float* const X = L.x + k * int64_t(n);
  const float inf = __builtin_inff();
  auto word_points = [&](int32_t word, float x[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = word < word1 && 4 * word + e < n ? X[4 * word + e] : inf;
  };
  float mine[4];
  word_points(word0 + int32_t(threadIdx.x), mine);
  const Cells g = cells_of(L.slots[slot_of(k)], D);
  count[2 * threadIdx.x] = count[2 * threadIdx.x + 1] = make_int4(0, 0, 0, 0);
  if (threadIdx.x == 0) run_column[0] = -inf;
  const int32_t samples = n < kSetSamples ? n : kSetSamples;
  float x[kLoads];
#pragma unroll
  for (int e = 0; e < kLoads; ++e) {
    const uint32_t q = uint32_t(e * kSetsBlock) + threadIdx.x;
    uint32_t i = q;
    // beyond kSetSamples: any one of the stretch's satellites (q n < 2^32)
    if (n > kSetSamples) i = ((q * uint32_t(n)) >> 14) + __umulhi(q * 0x9e3779b1u, uint32_t(n) >> 14);
    x[e] = int32_t(q) < samples ? X[i] : inf;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kLoads; ++e)
    if (x[e] < inf) atomicAdd(reinterpret_cast<int32_t*>(count) + strip_of(floorf(x[e] * g.inv_w)), 1);
  __syncthreads();

  // this lane's strips: their counts, the last count that is not zero, the points
  // before them and the last such count before them
  const int4 c0 = count[2 * threadIdx.x], c1 = count[2 * threadIdx.x + 1];
  const int32_t own[kOwn] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
  int32_t sum = 0, last = 0;
  float dense = 0.0f;
#pragma unroll
  for (int e = 0; e < kOwn; ++e) {
    sum += own[e];
    last = own[e] > 0 ? own[e] : last;
    dense += float(own[e]) * float(own[e] - 1);
  }
  dense /= strip_columns(kOwn * threadIdx.x);  // (the same for all eight)
  auto scan = [&](int32_t v, int lanes) {
    for (int o = 1; o < lanes; o <<= 1) {
      const int32_t u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    return v;
  };
  int32_t at = scan(sum, 64);
  const unsigned long long any = __ballot(last > 0);
  const unsigned long long lower = any & ((1ull << lane) - 1ull);
  int32_t prev = __shfl(last, lower ? 63 - __clzll(lower) : 0);
  const int32_t top = __shfl(last, any ? 63 - __clzll(any) : 0);
  for (int o = 32; o > 0; o >>= 1) dense += __shfl_xor(dense, o);
  if (lane == 63) {
    wave_points[wave] = at;
    wave_last[wave] = top;
    wave_dense[wave] = dense;
  }
  __syncthreads();
  const int32_t points = scan(wave_points[lane & 15], 16);
  const int32_t total = __shfl(points, 15), lasts = wave_last[lane & 15];
  at += (wave > 0 ? __shfl(points, wave - 1) : 0) - sum;
  {
    const unsigned long long m = __ballot(lane < wave && lasts > 0);
    const int32_t earlier = __shfl(lasts, m ? 63 - __clzll(m) : 0);
    if (!lower) prev = m ? earlier : 0;
  }
  float d = wave_dense[lane & 15];
  for (int o = 8; o > 0; o >>= 1) d += __shfl_xor(d, o);
  // the column around a point holds d / total of the counted ones, n / (2 l) for a
  // sphere of l columns radius
  const float all = float(n) * float(total) / float(samples);
  if (threadIdx.x == 0 && word0 == 0 && total > 0) {
    const float l = 0.5f * float(total) * float(total) / fmaxf(d, 1.0f);
    atomicMin(&L.slots[slot_of(k)].rows, __float_as_uint(row_widths(l, all)));
  }
  const int32_t runs = d * float(n) <= kTwoRunsColumn * float(total) * float(samples) ? 2 * slabs : slabs;
  // the strips that begin a run: another share at their middle than at the middle
  // of the strip before
  const float scale = 0.5f * float(runs) / float(total);
  uint32_t begin = 0;
#pragma unroll
  for (int e = 0; e < kOwn; ++e) {
    const bool differs = int32_t(float(2 * at + own[e]) * scale) != int32_t(float(2 * at - prev) * scale);
    if (own[e] > 0 && prev > 0 && differs) begin |= 1u << e;
    prev = own[e] > 0 ? own[e] : prev;
    at += own[e];
  }
  const int32_t begins = __popc(begin);
  int32_t number = scan(begins, 64);
  if (lane == 63) wave_begins[wave] = number;
  __syncthreads();
  const int32_t numbers = scan(wave_begins[lane & 15], 16);
  number += (wave > 0 ? __shfl(numbers, wave - 1) : 0) - begins;
  uint64_t eight = 0;
#pragma unroll
  for (int e = 0; e < kOwn; ++e) {
    if ((begin >> e) & 1u) run_column[++number] = strip_column(kOwn * threadIdx.x + e);
    eight |= uint64_t(uint32_t(number)) << (8 * e);
  }
  run_of[threadIdx.x] = eight;
  __syncthreads();

  const uint8_t* const run_of_strip = reinterpret_cast<const uint8_t*>(run_of);
  for (int32_t word = word0 + int32_t(threadIdx.x); word < word1; word += kSetsBlock) {
    float after[4];
    word_points(word + kSetsBlock, after);
    uint32_t out = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float c = floorf(mine[e] * g.inv_w);
      const uint32_t run = run_of_strip[mine[e] < inf ? strip_of(c) : 0u];
      const uint32_t set = run < uint32_t(slabs) ? run : run - uint32_t(slabs);
      const uint32_t v = run_column[run] == c ? set | 0x80u : set;
      out |= (mine[e] < inf ? v : 0xffu) << (8 * e);
      mine[e] = after[e];
    }
    L.cls[k * L.words + word] = out;
  }
}

// Points per table, hash heads, occupancy bits, pending walks and buffered
// events of a workgroup: 79 KiB of LDS, two workgroups (32 wavefronts) per
// compute unit.
constexpr int kSlabBlock = 1024;
constexpr int kSlabPoints = 3072;
constexpr int kSlabHeads = 2048;
constexpr int kSlabBits = 32768;
constexpr int kSlabWalks = 1536;
constexpr int kSlabEvents = 256;
static_assert(kSlabPoints <= 4096, "a pending walk holds 12 bits of entry and 2 of cell");
// Lanes of mask m below this one.
__device__ __forceinline__ int32_t rank_in(unsigned long long m) {
  return int32_t(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)));
}

// Work item u: sample time u / slabs and column set u % slabs.  Columns of width
// w > D + margins run over all x; a set is one or two runs of them.  A set's table
// holds its own points and, for the pairs across a run's upper edge, those of the
// next run's first column.  Each pair is met once: from its lower column, from its lower row
// within a column, once within a cell.  A set whose points exceed the table (all
// points in a few columns, say) takes the time's satellites in runs: a table per
// run, every own point of the time tested against each.
//
// The work: the stream of class bytes (every set reads its time's, five
// instructions for four points) and the cells' lookups.  One workgroup per time
// with a bucket sort by x in LDS took 219 us at 9,341 x 1,000, this kernel 123;
// buckets of x in device memory 2.6 ms for the sweep alone at 100,000 x 144, with
// 110 candidates per point, this kernel 0.48 ms.
//
// kOne: one set holds every point (n <= kSlabPoints): no classes, no overflow.
template <class TR, bool kOne>
__global__ void __launch_bounds__(kSlabBlock, 8)
    screen_slab_kernel(const TR* __restrict__ r, SlabLayout L, int32_t n, int64_t T, double D, double D2, int64_t cap,
                       int32_t slabs, int32_t* __restrict__ pairs, double* __restrict__ dist,
                       unsigned long long* __restrict__ count) {
  __shared__ float4 point[kSlabPoints];  // x, y, z and the chain's next entry
  __shared__ int32_t owner[kSlabPoints];  // satellite; ~satellite for the next runs' points
  __shared__ int32_t head[kSlabHeads];
  __shared__ uint32_t bits[kSlabBits / 32];  // cells (by a finer hash) that hold a point
  __shared__ uint16_t walks[kSlabWalks];
  __shared__ int2 event_pair[kSlabEvents];
  __shared__ double event_dist[kSlabEvents];
  __shared__ int32_t held, events, pending;
  __shared__ unsigned long long event_base;
  const int lane = threadIdx.x & 63;
  const int64_t P = int64_t(n) * T, total = T * slabs;
  // workgroup w runs on XCD w mod 8: each XCD takes a contiguous run of items,
  // so the workgroups of one time share an L2
  const int64_t per = (total + 7) / 8;
  for (int64_t v = blockIdx.x; v < 8 * per; v += gridDim.x) {
    const int64_t u = (v & 7) * per + (v >> 3);
    if ((v >> 3) >= per || u >= total) continue;  // uniform over the workgroup
    const int64_t k = u / slabs;
    const int32_t slab = int32_t(u - k * slabs);
    const float* const X = L.x + k * int64_t(n);
    const float* const Y = L.y + k * int64_t(n);
    const float* const Z = L.z + k * int64_t(n);

    const SlabSlot& slot = L.slots[slot_of(k)];
    const Cells g = cells_of(slot, D);
    const float near = g.near, near_z = g.near_z, reach = g.reach, inv_w = g.inv_w;
    const float inv_h = inv_w / (kOne ? row_widths(__uint_as_float(slot.rxy) * inv_w + 1.0f, float(n)) : __uint_as_float(slot.rows));
    auto column = [&](float x) { return column_of(x, inv_w); };
    auto row = [&](float y) { return int32_t(floorf(y * inv_h)); };
    // a cell's hash: its upper 11 bits are the head, its upper 15 the occupancy bit
    auto cell_hash = [&](int32_t c, int32_t b) { return uint32_t(c) * 0x9e3779b1u ^ uint32_t(b) * 0x85ebca77u; };
    auto bucket = [&](int32_t c, int32_t b) { return cell_hash(c, b) >> (32 - 11); };
    auto occupied = [&](int32_t c, int32_t b) {
      const uint32_t h = cell_hash(c, b) >> (32 - 15);
      return ((bits[h >> 5] >> (h & 31)) & 1u) != 0;
    };
    static_assert(kSlabHeads == 1 << 11 && kSlabBits == 1 << 15, "hash bits");
    // Table of the set's points among satellites [lo, hi), lo a multiple of four;
    // returns how many the class bytes name (past kSlabPoints none is stored).
    // The stream only notes which satellites belong; coordinates and chains are
    // left to full wavefronts afterwards.
    const uint32_t own_class = uint32_t(slab) * 0x01010101u;
    const uint32_t next_class = uint32_t((slab + 1) % slabs) * 0x01010101u;
    const uint32_t* const classes = L.cls + k * L.words;
    auto build = [&](int32_t lo, int32_t hi) {
      __syncthreads();
      for (int q = threadIdx.x; q < kSlabHeads; q += kSlabBlock) head[q] = -1;
      for (int q = threadIdx.x; q < kSlabBits / 32; q += kSlabBlock) bits[q] = 0u;
      if (threadIdx.x == 0) held = pending = 0;
      __syncthreads();
      const int32_t w1 = kOne ? 0 : (hi + 3) >> 2;
      for (int32_t w0 = lo >> 2; w0 < w1; w0 += 4 * kSlabBlock) {
        uint32_t word[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int32_t w = w0 + e * kSlabBlock + int32_t(threadIdx.x);
          word[e] = w < w1 ? classes[w] : 0xffffffffu;
        }
        // bit 8 b + e: point b of word e belongs (a byte of seven bits plus 0x7f
        // reaches bit 7 unless it is zero); above: those of a next run's first
        // column
        uint32_t flags = 0, above = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t low = word[e] & 0x7f7f7f7fu;
          const uint32_t own = ~((low ^ own_class) + 0x7f7f7f7fu), next = ~((low ^ next_class) + 0x7f7f7f7fu) & word[e];
          flags |= ((own | next) & 0x80808080u) >> (7 - e);
          above |= (next & 0x80808080u) >> (7 - e);
        }
        if (__ballot(flags != 0) == 0) continue;
        // places in the list: a prefix sum of the lanes' counts, bit by bit
        const int32_t mine = __popc(flags);
        int32_t before = 0, found = 0;
#pragma unroll
        for (int e = 0; e < 5; ++e) {
          const unsigned long long m = __ballot((mine >> e) & 1);
          if (m == 0) continue;
          before += rank_in(m) << e;
          found += __popcll(m) << e;
        }
        int32_t at = 0;
        if (lane == 0) at = atomicAdd(&held, found);
        at = __builtin_amdgcn_readfirstlane(at) + before;
        while (flags != 0) {
          const int f = __ffs(flags) - 1;
          flags &= flags - 1;
          const int32_t i = 4 * (w0 + (f & 7) * kSlabBlock + int32_t(threadIdx.x)) + (f >> 3);
          if (at < kSlabPoints) owner[at] = (above >> f) & 1u ? ~i : i;
          ++at;
        }
      }
      __syncthreads();
      const int32_t all = kOne ? n : held, m = all < kSlabPoints ? all : kSlabPoints;
      for (int32_t q = threadIdx.x; q < m; q += kSlabBlock) {
        const int32_t w = kOne ? q : owner[q], i = w < 0 ? ~w : w;
        const float x = X[i];
        if (kOne && !(x < __builtin_inff())) {
          owner[q] = ~i;  // invalid: in no chain, and takes no walks
          continue;
        }
        const int32_t c = column(x);
        const float y = Y[i], z = Z[i];
        const uint32_t h = cell_hash(c, row(y));
        atomicOr(&bits[h >> (32 - 10)], 1u << ((h >> (32 - 15)) & 31));
        const int32_t next = atomicExch(&head[h >> (32 - 11)], q);
        point[q] = make_float4(x, y, z, __int_as_float(next));
        if (kOne) owner[q] = i;
      }
      __syncthreads();
      return all;
    };

    auto report = [&](int32_t i, int32_t j, double d2) {
      const int32_t a = i < j ? i : j, b = i < j ? j : i;
      const double d = sqrt(d2);
      const int32_t e = atomicAdd(&events, 1);
      if (e < kSlabEvents) {
        event_pair[e] = make_int2(a, b);
        event_dist[e] = d;
      } else {
        // past the buffer: one addition for the lanes that report together
        const unsigned long long m = __ballot(1);
        const int32_t rank = rank_in(m);
        unsigned long long g = 0;
        if (rank == 0) g = atomicAdd(count, (unsigned long long)__popcll(m));
        g = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int32_t(g >> 32)))) << 32) |
            uint32_t(__builtin_amdgcn_readfirstlane(int32_t(g)));
        g += uint32_t(rank);
        if (int64_t(g) < cap) {
          pairs[3 * g] = a;
          pairs[3 * g + 1] = b;
          pairs[3 * g + 2] = int32_t(k);
          dist[g] = d;
        }
      }
    };

    // Candidates of point (x, y, z) of satellite i from entry q on along a chain,
    // in cell (c, b); after: only satellites after i (its own cell's pairs).
    auto walk = [&](int32_t q, int32_t c, int32_t b, bool after, float x, float y, float z, int32_t i) {
      while (q >= 0) {
        const float4 o = point[q];
        if (fabsf(o.x - x) <= near && fabsf(o.y - y) <= near && fabsf(o.z - z) <= near_z && column(o.x) == c &&
            row(o.y) == b) {
          const int32_t w = owner[q], j = w < 0 ? ~w : w;
          if (!after || j > i) {
            const double d2 = dist2(r, P, int64_t(i) * T + k, int64_t(j) * T + k);
            if (d2 < D2) report(i, j, d2);
          }
        }
        q = __float_as_int(o.w);
      }
    };
    // Walk e of table entry q: 0 its own chain from its next entry on (a pair in
    // one bucket is met once, from the later entry), 1 the cell above, 2 the next
    // column's cell, 3 that column's cell above or below, whichever is in reach
    // (a row is more than two reaches tall).
    auto table_walk = [&](int32_t q, int e) {
      const float4 o = point[q];
      const int32_t c = column(o.x), b = row(o.y), above = row(o.y + reach);
      const int32_t side = above != b ? above : row(o.y - reach);
      const int32_t cc = c + (e >> 1), bb = e == 0 || e == 2 ? b : e == 1 ? above : side;
      walk(e == 0 ? __float_as_int(o.w) : head[bucket(cc, bb)], cc, bb, false, o.x, o.y, o.z, owner[q]);
    };

    if (threadIdx.x == 0) events = 0;
    const int32_t m = build(0, n);
    if (kOne || m <= kSlabPoints) {
      // Most cells that could hold a partner are empty, and a wavefront that
      // walks chains for a few of its lanes takes as long as for all: so the
      // walks that the occupancy bits leave are listed first, then taken by full
      // wavefronts.
      const int32_t rounds = (m + kSlabBlock - 1) / kSlabBlock;
      for (int32_t t0 = 0; t0 < rounds; ++t0) {
        const int32_t q = t0 * kSlabBlock + threadIdx.x;
        bool go[4] = {false, false, false, false};
        if (q < m && owner[q] >= 0) {
          const float4 o = point[q];
          const int32_t c = column(o.x), b = row(o.y), above = row(o.y + reach);
          const int32_t side = above != b ? above : row(o.y - reach);
          go[0] = __float_as_int(o.w) >= 0;
          go[1] = above != b && occupied(c, above);
          go[2] = occupied(c + 1, b);
          go[3] = side != b && occupied(c + 1, side);
        }
        unsigned long long g[4];
        int32_t found = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          g[e] = __ballot(go[e]);
          found += __popcll(g[e]);
        }
        if (found == 0) continue;
        int32_t at = 0;
        if (lane == 0) at = atomicAdd(&pending, found);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (g[e] == 0) continue;
          const int32_t w = at + rank_in(g[e]);
          at += __popcll(g[e]);
          if (!go[e]) continue;
          if (w < kSlabWalks) walks[w] = uint16_t(q | (e << 12));
          else table_walk(q, e);
        }
      }
      __syncthreads();
      const int32_t listed = pending < kSlabWalks ? pending : kSlabWalks;
      for (int32_t w = threadIdx.x; w < listed; w += kSlabBlock) table_walk(walks[w] & 0xfff, walks[w] >> 12);
    } else {
      // runs of satellites whose points fit a table (runs of kSlabPoints always do)
      int32_t run = int32_t(int64_t(n) * kSlabPoints / (int64_t(m) * 5 / 4));
      run = (run < kSlabPoints ? kSlabPoints : run) & ~3;
      for (int32_t lo = 0; lo < n;) {
        const int32_t hi = n - lo < run ? n : lo + run;
        if (build(lo, hi) > kSlabPoints) {  // the same for all lanes
          run = (run / 2 < kSlabPoints ? kSlabPoints : run / 2) & ~3;
          continue;
        }
        lo = hi;
        for (int32_t w = threadIdx.x; w < int32_t(L.words); w += kSlabBlock) {
          const uint32_t word = classes[w];
          for (uint32_t f = ~(((word & 0x7f7f7f7fu) ^ own_class) + 0x7f7f7f7fu) & 0x80808080u; f != 0; f &= f - 1) {
            const int32_t i = 4 * w + ((__ffs(f) - 1) >> 3);
            const float x = X[i], y = Y[i], z = Z[i];
            const int32_t c = column(x), b = row(y), above = row(y + reach);
            const int32_t side = above != b ? above : row(y - reach);
            for (int e = 0; e < 4; ++e) {
              const int32_t cc = c + (e >> 1), bb = e == 0 || e == 2 ? b : e == 1 ? above : side;
              if ((e == 1 || e == 3) && bb == b) continue;
              walk(head[bucket(cc, bb)], cc, bb, e == 0, x, y, z, i);
            }
          }
        }
      }
    }
    __syncthreads();
    // the buffered events: one addition to the device counter per item
    const int32_t ne = events < kSlabEvents ? events : kSlabEvents;
    if (threadIdx.x == 0 && ne > 0) event_base = atomicAdd(count, (unsigned long long)ne);
    __syncthreads();
    for (int32_t e = threadIdx.x; e < ne; e += kSlabBlock) {
      const int64_t g = int64_t(event_base) + e;
      if (g < cap) {
        pairs[3 * g] = event_pair[e].x;
        pairs[3 * g + 1] = event_pair[e].y;
        pairs[3 * g + 2] = int32_t(k);
        dist[g] = event_dist[e];
      }
    }
    __syncthreads();
  }
}

__global__ void screen_clear(unsigned long long* count) {
  if (threadIdx.x == 0) *count = 0ull;
}

int screen_max_n() { return kScreenMaxN; }

// ---------------------------------------------------- device-memory path --
// A bucket sort of x in device memory and a sweep.  Buckets of x span a range [-R, R] with R the largest |x| of any valid point (one reduction over
// the batch), nb = n / 4 of them at most, width w >= D plus the rounding
// margin of R (fewer, wider buckets when the range is small).  Per time k:
// counts[k][b] (histogram, then offsets by an in-place scan, then ends after
// placement), and the sorted (x, y) and satellite index of the valid points.
struct GHeader {
  unsigned int rbits;  // largest valid |x| as float bits (non-negative floats order as integers)
  int32_t nb;          // buckets in use per time
  double x0, inv_w;    // bucket b = (x - x0) * inv_w
};

struct GLayout {
  GHeader* hdr;
  int32_t* counts;  // [T][nbmax + 1]
  float2* sxy;      // [T][n]
  int32_t* sidx;    // [T][n]
  int64_t nbmax;
};

static int64_t screen_global_buckets(int64_t n) {
  int64_t nb = n / 4;
  if (nb < 16) nb = 16;
  if (nb > (int64_t(1) << 20)) nb = int64_t(1) << 20;
  return nb;
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

static GLayout global_layout(void* ws, int64_t n, int64_t T) {
  GLayout L;
  L.nbmax = screen_global_buckets(n);
  char* b = static_cast<char*>(ws);
  L.hdr = reinterpret_cast<GHeader*>(b);
  b += align256(sizeof(GHeader));
  L.counts = reinterpret_cast<int32_t*>(b);
  b += align256(size_t(T) * size_t(L.nbmax + 1) * 4);
  L.sxy = reinterpret_cast<float2*>(b);
  b += align256(size_t(T) * size_t(n) * 8);
  L.sidx = reinterpret_cast<int32_t*>(b);
  return L;
}

static size_t global_ws_bytes(int64_t n, int64_t T) {
  const int64_t nbmax = screen_global_buckets(n);
  return align256(sizeof(GHeader)) + align256(size_t(T) * size_t(nbmax + 1) * 4) + align256(size_t(T) * size_t(n) * 8) +
         size_t(T) * size_t(n) * 4;
}

template <class TR>
__device__ __forceinline__ bool valid_point(const TR* __restrict__ r, const uint8_t* __restrict__ err, int64_t P,
                                            int64_t p, float* x, float* y) {
  const TR vx = r[p], vy = r[P + p], vz = r[2 * P + p];
  bool ok = isfinite(double(vx)) && isfinite(double(vy)) && isfinite(double(vz));
  if (err) ok = ok && (err[p] == 0 || err[p] == 6);
  *x = float(vx);
  *y = float(vy);
  return ok;
}

// Clear the header and the counts (a fill kernel, so the launch sequence can
// be captured in a graph).
__global__ void gscreen_clear(GLayout L, int64_t T) {
  const int64_t total = T * (L.nbmax + 1);
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < total; q += int64_t(gridDim.x) * blockDim.x)
    L.counts[q] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    L.hdr->rbits = 0u;
    L.hdr->nb = 0;
  }
}

template <class TR>
__global__ void __launch_bounds__(256) gscreen_range(const TR* __restrict__ r, const uint8_t* __restrict__ err,
                                                     int64_t P, GLayout L) {
  float m = 0.0f;
  for (int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x; p < P; p += int64_t(gridDim.x) * 256) {
    float x, y;
    if (valid_point(r, err, P, p, &x, &y)) m = fmaxf(m, fabsf(x));
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  // one address for the whole batch: an atomic takes ~11 ns, so one per
  // workgroup of a grid that just fills the chip (one per wavefront of 16,384
  // workgroups took 754 us at 100,000 x 144)
  __shared__ float wave_max[4];
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(&L.hdr->rbits,
              __float_as_uint(fmaxf(fmaxf(wave_max[0], wave_max[1]), fmaxf(wave_max[2], wave_max[3]))));
}

__global__ void gscreen_buckets(GLayout L, double D) {
  if (threadIdx.x != 0) return;
  const double R = double(__uint_as_float(L.hdr->rbits));
  const double span = 2.0 * R;
  const double w = fmax((D + 2.4e-7 * R) * (1.0 + 1.0e-6), span / double(L.nbmax - 1));
  int64_t nb = int64_t(span / w) + 1;
  if (nb > L.nbmax) nb = L.nbmax;
  L.hdr->nb = int32_t(nb);
  L.hdr->x0 = -R;
  L.hdr->inv_w = 1.0 / w;
}

__device__ __forceinline__ int32_t gbucket(const GHeader& h, float x) {
  const int32_t b = int32_t((double(x) - h.x0) * h.inv_w);
  return b < h.nb - 1 ? b : h.nb - 1;
}

template <class TR>
__global__ void __launch_bounds__(256) gscreen_count(const TR* __restrict__ r, const uint8_t* __restrict__ err,
                                                     int64_t T, int64_t P, GLayout L) {
  const GHeader h = *L.hdr;
  const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= P) return;
  float x, y;
  if (!valid_point(r, err, P, p, &x, &y)) return;
  const int64_t k = p % T;
  atomicAdd(&L.counts[k * (L.nbmax + 1) + gbucket(h, x) + 1], 1);
}

// Inclusive scan of counts[k][1..nb] per time (one workgroup per time, 256
// lanes, chunks of 256 buckets with a running carry).
__global__ void __launch_bounds__(256) gscreen_scan(GLayout L) {
  __shared__ int32_t part[4];
  __shared__ int32_t carry_s;
  const int32_t nb = L.hdr->nb;
  int32_t* c = L.counts + int64_t(blockIdx.x) * (L.nbmax + 1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t carry = 0;
  for (int32_t base = 1; base <= nb; base += 256) {
    const int32_t b = base + int32_t(threadIdx.x);
    int32_t v = b <= nb ? c[b] : 0;
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t u = __shfl_up(v, o);
      if (lane >= o) v += u;
    }
    if (lane == 63) part[wave] = v;
    __syncthreads();
    int32_t before = carry;
    for (int q = 0; q < wave; ++q) before += part[q];
    if (b <= nb) c[b] = before + v;
    if (threadIdx.x == 255) carry_s = before + v;
    __syncthreads();
    carry = carry_s;
    __syncthreads();
  }
}

template <class TR>
__global__ void __launch_bounds__(256) gscreen_place(const TR* __restrict__ r, const uint8_t* __restrict__ err,
                                                     int64_t n, int64_t T, GLayout L) {
  const GHeader h = *L.hdr;
  const int64_t P = n * T;
  const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (p >= P) return;
  float x, y;
  if (!valid_point(r, err, P, p, &x, &y)) return;
  const int64_t i = p / T, k = p - (p / T) * T;
  const int32_t q = atomicAdd(&L.counts[k * (L.nbmax + 1) + gbucket(h, x)], 1);
  L.sxy[k * n + q] = make_float2(x, y);
  L.sidx[k * n + q] = int32_t(i);
}

template <class TR>
__global__ void __launch_bounds__(256)
    gscreen_sweep(const TR* __restrict__ r, int64_t n, int64_t T, double D, double D2, GLayout L, int64_t cap,
                  int32_t* __restrict__ pairs, double* __restrict__ dist, unsigned long long* __restrict__ count) {
  const GHeader h = *L.hdr;
  const int64_t g = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (g >= n * T) return;
  const int64_t k = g / n, q = g - (g / n) * n;
  const int32_t* c = L.counts + k * (L.nbmax + 1);
  if (q >= c[h.nb - 1]) return;  // after placement c[b] is the end of bucket b
  const float2* sxy = L.sxy + k * n;
  const int32_t* sidx = L.sidx + k * n;
  const int64_t P = n * T;
  const float2 vi = sxy[q];
  const int32_t i = sidx[q];
  const int32_t b = gbucket(h, vi.x);
  const int32_t end = b + 1 < h.nb ? c[b + 1] : c[b];
  const double xi = vi.x, yi = vi.y;
  const int64_t pi = int64_t(i) * T + k;
  // candidates in groups of eight: the group's loads are issued together (a
  // position past the bucket's end reads as NaN and fails the tests)
  constexpr int kU = 8;
  for (int32_t q0 = int32_t(q) + 1; q0 < end; q0 += kU) {
    float2 vj[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      vj[u] = q0 + u < end ? sxy[q0 + u] : make_float2(__builtin_nanf(""), __builtin_nanf(""));
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const double xj = vj[u].x, yj = vj[u].y;
      if (!(fabs(xj - xi) < D + 1.2e-7 * (fabs(xi) + fabs(xj)))) continue;
      if (!(fabs(yj - yi) < D + 1.2e-7 * (fabs(yi) + fabs(yj)))) continue;
      const int32_t j = sidx[q0 + u];
      const int64_t pj = int64_t(j) * T + k;
      const double d2 = dist2(r, P, pi, pj);
      if (d2 < D2) {
        const unsigned long long e = atomicAdd(count, 1ull);
        if (int64_t(e) < cap) {
          pairs[3 * e] = i < j ? i : j;
          pairs[3 * e + 1] = i < j ? j : i;
          pairs[3 * e + 2] = int32_t(k);
          dist[e] = sqrt(d2);
        }
      }
    }
  }
}

template <class TR>
static hipError_t screen_global(const TR* r, const uint8_t* err, int64_t n, int64_t T, double D, int64_t cap,
                                int32_t* pairs, double* dist, unsigned long long* count, void* ws, hipStream_t s) {
  const GLayout L = global_layout(ws, n, T);
  const int64_t P = n * T;
  const unsigned gp = unsigned((P + 255) / 256);
  const int64_t cells = T * (L.nbmax + 1);
  hipLaunchKernelGGL(gscreen_clear, dim3(unsigned(std::min<int64_t>((cells + 255) / 256, 65536))), dim3(256), 0, s,
                     L, T);
  hipLaunchKernelGGL(gscreen_range<TR>, dim3(unsigned(std::min<int64_t>((P + 255) / 256, 2048))), dim3(256), 0, s,
                     r, err, P, L);
  hipLaunchKernelGGL(gscreen_buckets, dim3(1), dim3(64), 0, s, L, D);
  hipLaunchKernelGGL(gscreen_count<TR>, dim3(gp), dim3(256), 0, s, r, err, T, P, L);
  hipLaunchKernelGGL(gscreen_scan, dim3(unsigned(T)), dim3(256), 0, s, L);
  hipLaunchKernelGGL(gscreen_place<TR>, dim3(gp), dim3(256), 0, s, r, err, n, T, L);
  hipLaunchKernelGGL(gscreen_sweep<TR>, dim3(gp), dim3(256), 0, s, r, n, T, D, D * D, L, cap, pairs, dist, count);
  return hipGetLastError();
}

// Catalogues beyond this take the device-memory path: every column set streams
// the whole time's class bytes, which grows with the square of n, and a class
// byte numbers up to 127 sets (0x7f is left to invalid points).
constexpr int64_t kSlabMaxN = 200000;

// Workspace of the two paths: the larger one's, the device-memory path's (the
// header, the per-time bucket offsets and 12 bytes per point).  The column path
// counts where it can be taken only: beyond four million satellites, where the
// buckets stop growing, its layout would be the larger one.
size_t screen_ws_bytes(int64_t n, int64_t T) {
  const size_t slab = n <= kSlabMaxN ? slab_ws_bytes(n, T) : 0;
  const size_t glob = global_ws_bytes(n, T);
  return slab > glob ? slab : glob;  // enough for either path
}

// Largest n * T the device-memory path indexes (grids of 256-lane workgroups).
bool screen_global_fits(int64_t n, int64_t T) {
  return n <= 0x7fffffff && n * T <= int64_t(0x7fffffff) * 256 && T <= 0x7fffffff;
}

// Column sets per time: about 2,050 points each, less for larger catalogues (a
// sixth at 200,000 satellites, whose shares are sampled and whose columns hold
// more).  A table of 3,072 then has room for half a strip at either end of a run
// and the column above: the fullest set of shells at 10 km holds 1,890 to 2,450
// points from 9,341 to 200,000 satellites and, at 100 km, about 3,000 of 100,000,
// also with single satellites at 42,164, 120,000 or 4e6 km or one in twenty on the
// geostationary ring (2,400 each overflowed there from 50,000 satellites on).  A set
// that overflows (a column of its own with more than 3,072 points, say) works in
// runs of satellites.
static int32_t slab_count(int64_t n) {
  return n <= kSlabPoints ? 1 : int32_t((n + n * n / 1000000 + 2047) / 2048);
}

template <class TR>
static hipError_t screen_slabs(const TR* r, const uint8_t* err, int64_t n, int64_t T, double D, int64_t cap,
                               int32_t* pairs, double* dist, unsigned long long* count, void* ws, hipStream_t s) {
  const SlabLayout L = slab_layout(ws, n, T);
  const int32_t slabs = slab_count(n);
  hipLaunchKernelGGL(slab_clear, dim3(1), dim3(64), 0, s, L, count);
  hipLaunchKernelGGL(screen_pack<TR>, dim3(unsigned((T + 63) / 64), unsigned((n + 63) / 64)), dim3(256), 0, s, r, err,
                     n, T, L);
  const int64_t items = (T * slabs + 7) / 8 * 8;
  const dim3 grid(unsigned(std::min<int64_t>(items, (int64_t(1) << 32) / kSlabBlock - 8)));
  if (slabs == 1) {
    hipLaunchKernelGGL((screen_slab_kernel<TR, true>), grid, dim3(kSlabBlock), 0, s, r, L, int32_t(n), T, D, D * D,
                       cap, slabs, pairs, dist, count);
  } else {
    // workgroups per time: as many as fill the chip once (two on a compute unit;
    // each counts the time's points anew), with a class word per lane at least
    const int64_t parts = std::max<int64_t>(1, std::min((L.words + kSetsBlock - 1) / kSetsBlock, 512 / T));
    const int64_t part_words = (L.words + parts - 1) / parts;
    hipLaunchKernelGGL(screen_sets, dim3(unsigned(T * parts)), dim3(kSetsBlock), 0, s, L, int32_t(n), T, D, slabs,
                       int32_t(parts), int32_t(part_words));
    hipLaunchKernelGGL((screen_slab_kernel<TR, false>), grid, dim3(kSlabBlock), 0, s, r, L, int32_t(n), T, D, D * D,
                       cap, slabs, pairs, dist, count);
  }
  return hipGetLastError();
}

// mode 0: the column path up to kSlabMaxN satellites, else the device-memory
// path; 1: the column path (the caller checks n); 2: the device-memory path.
hipError_t launch_screen(const void* r, bool fp64, const uint8_t* err, int64_t n, int64_t T, double D, int64_t cap,
                         int32_t* pairs, double* dist, unsigned long long* count, void* ws, int mode, hipStream_t s) {
  const bool global = mode == 2 || (mode == 0 && n > kSlabMaxN);
  if (n < 2 || T == 0 || global) {
    hipLaunchKernelGGL(screen_clear, dim3(1), dim3(64), 0, s, count);
    if (n < 2 || T == 0) return hipGetLastError();
  }
  if (global) {
    if (fp64) return screen_global(static_cast<const double*>(r), err, n, T, D, cap, pairs, dist, count, ws, s);
    return screen_global(static_cast<const float*>(r), err, n, T, D, cap, pairs, dist, count, ws, s);
  }
  if (fp64) return screen_slabs(static_cast<const double*>(r), err, n, T, D, cap, pairs, dist, count, ws, s);
  return screen_slabs(static_cast<const float*>(r), err, n, T, D, cap, pairs, dist, count, ws, s);
}

// ------------------------------------------------------------- no-alloc --
// Workspace for callers that cannot allocate device memory: a fixed array in
// the code object, one copy per GPU the library runs on, held until the
// process ends.  Host code never passes `scratch` itself to a kernel (on the
// host it names a stand-in, not device memory); it passes the device address
// taken with hipGetSymbolAddress once per device, with that device current.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t screen_static_bytes() { return kStaticScratchBytes; }

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// This GPU's copy of the scratch array (the current device's), looked up on
// the first call on that device.
static hipError_t scratch_of_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// launch_screen (mode 0) with the workspace in this GPU's scratch array; the
// caller checks that screen_ws_bytes(n, T) fits kStaticScratchBytes.  Both
// paths initialise every workspace byte they read (the packing pass writes
// all n T entries; the device-memory path clears its header and counts with a
// kernel), so nothing of an earlier call's contents is used.
hipError_t launch_screen_static(const void* r, bool fp64, const uint8_t* err, int64_t n, int64_t T, double D,
                                int64_t cap, int32_t* pairs, double* dist, unsigned long long* count, hipStream_t s) {
  void* ws = nullptr;
  if (hipError_t e = scratch_of_current_device(&ws)) return e;
  return launch_screen(r, fp64, err, n, T, D, cap, pairs, dist, count, ws, 0, s);
}

}  // namespace sgp4mi
