// prefill.hip -- preparation of the prefill grouped GEMMs (expert tile tables
// and the bf16 fragment-tiled copy of the routed token rows, in one launch)
// and their launcher.  The GEMM kernels are in prefill.hpp, one file per
// group size.
#include "prefill.hpp"
#include "route_device.hpp"
#include <algorithm>

namespace mc {

extern template hipError_t launch_prefill_gemm<1>(const LayerArgs&, const int32_t*, const PrefillTables&,
                                                  const PrefillGemm&, bool, int, hipStream_t);
extern template hipError_t launch_prefill_gemm<2>(const LayerArgs&, const int32_t*, const PrefillTables&,
                                                  const PrefillGemm&, bool, int, hipStream_t);
extern template hipError_t launch_prefill_gemm<4>(const LayerArgs&, const int32_t*, const PrefillTables&,
                                                  const PrefillGemm&, bool, int, hipStream_t);

// The prefill's preparation, one workgroup per fragment row f (f_max of them)
// and block of kGatherCols columns.  Every workgroup first scans the expert
// counts itself (thread e: fragment rows ceil(M_e/32) and m-tiles of tb.tiles
// fragment rows; wave prefix sums), which gives the expert that f belongs to;
// the first one also writes the tables the GEMMs read.  Counts outside [0, P]
// are taken as 0, and tables that would not fit their capacity are left empty
// (no m-tiles, no fragment rows), so inconsistent routing cannot make any later
// access leave its buffer.
// Then the block of f's 32 routed rows of x (zero past the expert's count) is
// copied into the fragment layout (bf16, unchanged), with the sum of each group
// of G columns of each row in fp32: each wave reads whole rows of the block (64
// lanes x 16 consecutive bytes) into a row-major LDS tile and forms the group
// sums of its pieces (the GP = G/8 lanes of a group add with the DPP butterfly of
// the decode slabs); then the workgroup writes the block's fragments
// (contiguous in the fragment layout) from the tile with consecutive 16-byte
// stores.
constexpr int kGatherThreads = 256;
constexpr int kGatherCols = 512;                     // columns of a block: 8 per lane
constexpr int kGatherStride = kGatherCols + 8;       // LDS row stride (elements): rows start on different banks

template <int GP>
__global__ void __launch_bounds__(kGatherThreads) prefill_prep_kernel(const uint16_t* __restrict__ x, int d, int E,
                                                                      const int32_t* __restrict__ counts,
                                                                      const int32_t* __restrict__ offsets,
                                                                      const int32_t* __restrict__ pair_token,
                                                                      PrefillTables tb, uint16_t* __restrict__ xt,
                                                                      float* __restrict__ xsum) {
  static_assert(kPfFragRows * kGatherStride * 2 <= 64 * 1024, "gather tile");
  static_assert(kGatherThreads >= MC_MAX_EXPERTS, "a thread per expert");
  constexpr int kWaves = kGatherThreads / 64;
  __shared__ __attribute__((aligned(16))) uint16_t tile[kPfFragRows * kGatherStride];
  __shared__ int wf[kWaves], wm[kWaves], s_e, s_fb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int f = blockIdx.x;

  // tables: exclusive prefix sums of the experts' fragment rows and m-tiles
  const int c = tid < E ? checked_count(counts[tid], tb.P) : 0;
  const int nf = (c + kPfFragRows - 1) / kPfFragRows;
  const int nm = (nf + tb.tiles - 1) / tb.tiles;
  int sf = nf, sm = nm;
  for (int off = 1; off < 64; off <<= 1) {
    const int a = __shfl_up(sf, off), b = __shfl_up(sm, off);
    if (lane >= off) {
      sf += a;
      sm += b;
    }
  }
  if (lane == 63) {
    wf[wave] = sf;
    wm[wave] = sm;
  }
  __syncthreads();
  int tf = 0, tm = 0, fb = sf - nf, mb = sm - nm;
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) {
      fb += wf[w];
      mb += wm[w];
    }
    tf += wf[w];
    tm += wm[w];
  }
  const bool fits = tf <= tb.f_max && tm <= tb.mt_max;
  if (f == 0 && blockIdx.y == 0) {
    if (!fits) {
      for (int i = tid; i <= E; i += kGatherThreads) tb.ftile_base[i] = 0;
      if (tid == 0) *tb.mt_count = 0;
    } else {
      if (tid < E) {
        tb.ftile_base[tid] = fb;
        for (int i = 0; i < nm; ++i) {
          tb.mt_e[mb + i] = tid;
          tb.mt_j[mb + i] = i;
        }
      }
      if (tid == 0) {
        tb.ftile_base[E] = tf;
        *tb.mt_count = tm;
      }
    }
  }
  if (!fits || f >= tf) return;   // workgroup-uniform
  if (tid < E && fb <= f && f < fb + nf) {   // exactly one expert holds f
    s_e = tid;
    s_fb = fb;
  }
  __syncthreads();
  const int e = s_e;
  int ebase, ecount;
  expert_range_offsets(offsets, e, tb.P, ebase, ecount);
  const int pos0 = ebase + (f - s_fb) * kPfFragRows;
  const int pend = ebase + ecount;
  constexpr int kRowsPerWave = kPfFragRows / (kGatherThreads / 64);
  // this wave's rows: m = wave + 4 j; their token rows of x (past the list: row 0,
  // read and dropped, so that every load goes out before the first use; behind
  // branches each waited for the one before it: Mixtral layer, 4096 tokens, 26 us
  // -> 47)
  const uint16_t* src[kRowsPerWave];
#pragma unroll
  for (int j = 0; j < kRowsPerWave; ++j) {
    const int pos = pos0 + wave + 4 * j;
    src[j] = x + (size_t)(pos < pend ? clamp_token(pair_token[pos], tb.T) : 0) * d;
  }
  const int ng = d / (8 * GP);
  unsigned char* out = reinterpret_cast<unsigned char*>(xt) + frag_offset(f, 0, 0, d);
  const int c0 = blockIdx.y * kGatherCols;
  const int w = (d - c0) < kGatherCols ? (d - c0) : kGatherCols;   // a multiple of 128
  const bool on = 8 * lane < w;
  u32x4 v[kRowsPerWave];
#pragma unroll
  for (int j = 0; j < kRowsPerWave; ++j)
    v[j] = *reinterpret_cast<const u32x4*>(src[j] + c0 + (on ? 8 * lane : 0));
#pragma unroll
  for (int j = 0; j < kRowsPerWave; ++j)
    if (pos0 + wave + 4 * j >= pend) v[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < kRowsPerWave; ++j) {
    const int m = wave + 4 * j;
    if (on) *reinterpret_cast<u32x4*>(tile + m * kGatherStride + 8 * lane) = v[j];
    const float sum = lane_group_sum<GP>(sum8<false>(v[j]));
    if (on && lane % GP == 0) xsum[((size_t)f * ng + (c0 + 8 * lane) / (8 * GP)) * 32 + m] = sum;
  }
  __syncthreads();
  // fragment fi of the block, piece mm: row mm % 32, columns 16 fi + 8 (mm / 32)
  const int pieces = (w / 16) * 64;
  for (int p = threadIdx.x; p < pieces; p += kGatherThreads) {
    const int fi = p >> 6, mm = p & 63;
    *reinterpret_cast<u32x4*>(out + ((size_t)(c0 / 16 + fi) * 64 + mm) * 16) =
        *reinterpret_cast<const u32x4*>(tile + (mm & 31) * kGatherStride + 16 * fi + 8 * (mm >> 5));
  }
}

// Routing and preparation in one launch, for batches that one workgroup
// routes: every workgroup (fragment row f, block of kGatherCols columns) routes
// the whole batch in its LDS (a few us that a launch of its own would take too,
// and its results are at hand: no second launch, no tables to read back), takes
// f's rows from the experts' token masks and gathers its block as
// prefill_prep_kernel does; the first workgroup publishes the routing and the
// GEMMs' tables.  Tiny layer (4 experts), 64 tokens: 4.8 + 5.0 us in two
// launches, 6.9 in one, 24.4 -> 21.4 a call; Mixtral layer (8), 64 tokens: 5.6 +
// 6.3 and 7.6.  With many experts the selection is long and the fragment rows
// many, two workgroups a CU: OLMoE layer (64), 16 tokens: 7.8 + 5.5 us in two
// launches, 13.8 in one, so those keep them.
template <int GP>
__global__ void __launch_bounds__(64 * kRouteWaves) route_prep_kernel(
    const float* __restrict__ logits, const uint8_t* __restrict__ important, int T, int E, int k, float delta32,
    double tau, RouteBufs o, const uint16_t* __restrict__ x, int d, PrefillTables tb, uint16_t* __restrict__ xt,
    float* __restrict__ xsum) {
  static_assert(kPfFragRows * kGatherStride * 2 <= kRouteWaves * kSelScratchBytes, "the gather tile reuses the scratch");
  static_assert(kPfFragRows == 2 * kRouteWaves, "two rows a wave");
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int f = blockIdx.x;
  const bool first = blockIdx.x == 0 && blockIdx.y == 0;
  const RouteSmall s = route_small_batch(logits, important, T, E, k, delta32, tau, o, first);
  __syncthreads();
  // tables: lane e of every wave holds expert e (prefill_routes: E <= 16)
  const int nf = lane < E ? (s.lists.cnt[lane] + kPfFragRows - 1) / kPfFragRows : 0;
  const int nm = (nf + tb.tiles - 1) / tb.tiles;
  int sf = nf, sm = nm;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int a = __shfl_up(sf, off), b = __shfl_up(sm, off);
    if (lane >= off) {
      sf += a;
      sm += b;
    }
  }
  const int tf = __builtin_amdgcn_readlane(sf, 63), fb = sf - nf, mb = sm - nm;
  if (first && wave == 0) {
    if (lane < E) {
      tb.ftile_base[lane] = fb;
      for (int i = 0; i < nm; ++i) {
        tb.mt_e[mb + i] = lane;
        tb.mt_j[mb + i] = i;
      }
    }
    if (lane == 63) {
      tb.ftile_base[E] = sf;
      *tb.mt_count = sm;
    }
  }
  if (f >= tf) return;   // workgroup-uniform
  const int e = __builtin_ctzll(__ballot(fb <= f && f < fb + nf));   // exactly one expert holds f
  const int r0 = kPfFragRows * (f - __builtin_amdgcn_readlane(fb, e));
  // lane t: token t's place in e's list
  const unsigned long long mask = s.lists.bal[e];
  const bool on_list = (mask >> lane) & 1ull;
  const int place = __popcll(mask & ((1ull << lane) - 1ull));
  const int c0 = blockIdx.y * kGatherCols;
  const int w = (d - c0) < kGatherCols ? (d - c0) : kGatherCols;   // a multiple of 128
  const bool on = 8 * lane < w;
  const int ng = d / (8 * GP);
  uint16_t* tile = reinterpret_cast<uint16_t*>(s.scratch);   // the selections are done
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = 2 * wave + j;
    const unsigned long long who = __ballot(on_list && place == r0 + m);
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (on && who) v = *reinterpret_cast<const u32x4*>(x + (size_t)__builtin_ctzll(who) * d + c0 + 8 * lane);
    if (on) *reinterpret_cast<u32x4*>(tile + m * kGatherStride + 8 * lane) = v;
    const float sum = lane_group_sum<GP>(sum8<false>(v));
    if (on && lane % GP == 0) xsum[((size_t)f * ng + (c0 + 8 * lane) / (8 * GP)) * 32 + m] = sum;
  }
  __syncthreads();
  unsigned char* out = reinterpret_cast<unsigned char*>(xt) + frag_offset(f, 0, 0, d);
  const int pieces = (w / 16) * 64;
  for (int p = threadIdx.x; p < pieces; p += 64 * kRouteWaves) {
    const int fi = p >> 6, mm = p & 63;
    *reinterpret_cast<u32x4*>(out + ((size_t)(c0 / 16 + fi) * 64 + mm) * 16) =
        *reinterpret_cast<const u32x4*>(tile + (mm & 31) * kGatherStride + 16 * fi + 8 * (mm >> 5));
  }
}

bool prefill_routes(int T, int E) { return E <= 16 && route_fused_fits(T, E); }

static size_t round256(size_t b) { return ((b + 255) / 256) * 256; }

// The most m-tiles of a batch: every expert's last one may be short.
static int prefill_mt_max(int tiles, int T, int E, int k) {
  const size_t mtok = (size_t)tiles * kPfFragRows;
  return (int)(((size_t)T * k + (mtok - 1) * E) / mtok);
}

// The most splits of the down reduction: at least 8 chunks in each.
static int prefill_most_splits(int ffn) {
  const int most = (ffn / kTileCols) / 8;
  return most < 1 ? 1 : most < 4 ? most : 4;
}

// Fragment rows of the m-tiles.  Larger m-tiles unpack (and read) the weights
// less often, smaller ones keep more workgroups on a CU and leave less padding
// and a shorter last round, so the choice follows the pairs an expert sees and
// the gate/up workgroups that 64-token m-tiles would give.  Measured (us a layer
// call, m-tiles of 1 / 2 / 4 fragment rows):
//   Mixtral layer (G = 128): 64 tokens 151 / 160 / 237, 128: 190 / 187 / 267,
//     200: 251 / 233 / 289, 333: 355 / 305 / 409, 1200: - / 834 / 890; G = 64,
//     1024 tokens: - / 884 / 921, 4096: - / 3110 / 2930
//   OLMoE layer (G = 64): 512 tokens 120 / 125 / 163, 1024: 189 / 187 / 225,
//     2048: 321 / 316 / 358
//   60 experts of 2432 x 2944: 256 tokens 141 / 178 / -, 700: 183 / 202 / 272
//   tiny layer (256 x 512): 400 tokens 28 / 31 / 46, 2401: 39 / 42 / 53
//   8 experts of 256 x 9216: 300 tokens 55 / 61 / 102, 800: 84 / 81 / 128,
//     4096: 308 / 266 / 306
// The 128-token ones pay off for long reductions and grids of many rounds only:
// in a short run the 64-token ones are faster there too (Mixtral, 4096 tokens:
// 2468 against 2573 us), but under sustained load, where the card's power sets
// the clock, the extra unpacking costs more than it hides (2889 against 2867).
// A launch holds fewer than 2^32 threads, four a row of gate/up and two a row
// of down: where small m-tiles would need more, larger ones are taken.
static int prefill_tiles(int T, int E, int k, int d, int ffn) {
  const double per = (double)T * k / E;
  const double wgs2 = E * (per / 64 + 0.5) * ffn / 128;     // gate/up workgroups of 64-token m-tiles
  int tiles = per >= 512 && wgs2 >= 7000 && d >= 2048 && ffn >= 2048 ? 4 : 2;
  if (per <= 36 || wgs2 < 1000) tiles = 1;
  const double threads = std::max(4.0 * ffn, 2.0 * (d + 256.0) * prefill_most_splits(ffn));   // of an m-tile
  while (tiles < 4 && prefill_mt_max(tiles, T, E, k) * threads >= 4294967296.0) tiles *= 2;
  return tiles;
}

// Weight rows of a workgroup (ffn rows of gate/up, d rows of down).
template <int GPC>
static int prefill_rows_g(int tiles, bool gateup) {
  if (tiles == 1) return gateup ? PfTile<1, GPC>::kRowsGateUp : PfTile<1, GPC>::kRowsDown;
  if (tiles == 2) return gateup ? PfTile<2, GPC>::kRowsGateUp : PfTile<2, GPC>::kRowsDown;
  return gateup ? PfTile<4, GPC>::kRowsGateUp : PfTile<4, GPC>::kRowsDown;
}
static int prefill_rows(int tiles, int G, bool gateup) {
  return G == 128 ? prefill_rows_g<1>(tiles, gateup) : G == 64 ? prefill_rows_g<2>(tiles, gateup)
                                                               : prefill_rows_g<4>(tiles, gateup);
}

// What the down reduction's splits follow: its row blocks, the workgroups at
// once and the most splits.
struct PrefillSplit {
  int tiles, nt_down, slots, most;
};
static PrefillSplit prefill_split(int tiles, int d, int ffn, int G) {
  const int rows = prefill_rows(tiles, G, false);
  return {tiles, (d + rows - 1) / rows, 256 * (tiles == 4 ? 1 : tiles == 2 ? (G == 128 ? 2 : 3) : 4),
          prefill_most_splits(ffn)};
}

// The m-tiles that the splits are chosen for: the small tiles' count is about
// those in use.
static long long prefill_mt_planned(int tiles, int T, int E, int k) {
  const long long mt = prefill_mt_max(tiles, T, E, k);
  if (tiles == 4) return mt;
  const double per = (double)T * k / E / (tiles * kPfFragRows);
  const long long est = (long long)(E * (per < 0.5 ? 1.0 : per + 0.5));
  return est < mt ? est : mt;
}

// Splits of the down GEMM's reduction, so that its workgroups fill the CUs in
// whole rounds: the s minimising rounds(s) / s (the time of one round shrinks
// as 1/s), the smallest on ties.  It depends on mt * nt_down modulo the slots
// only.
static int prefill_nsplit(const PrefillSplit& p, long long mt) {
  const long long wgs = mt * p.nt_down;
  int s = 1;
  for (int c = 2; c <= p.most; ++c)
    if ((double)((wgs * c + p.slots - 1) / p.slots) / c < (double)((wgs * s + p.slots - 1) / p.slots) / s - 1e-9) s = c;
  return s;
}

// The layout with no down partials yet (total = part).
static PrefillLayout prefill_layout_base(int tiles, int T, int E, int k, int d, int ffn) {
  PrefillLayout pl;
  const size_t P = (size_t)T * k;
  pl.f_max = (int)((P + (size_t)(kPfFragRows - 1) * E) / kPfFragRows);
  pl.tiles = tiles;
  pl.mt_max = prefill_mt_max(tiles, T, E, k);
  // the GEMMs stage whole m-tiles: tiles - 1 padding fragment rows past the last one
  const size_t rows = (size_t)(pl.f_max + pl.tiles) * kPfFragRows;
  pl.tables = 0;
  const size_t tab = (size_t)(E + 1 + 2 * pl.mt_max + 1) * sizeof(int32_t);
  pl.x = round256(tab);
  pl.xsum = pl.x + round256(rows * d * sizeof(uint16_t));
  pl.h = pl.xsum + round256(rows * (d / 32) * sizeof(float));   // G >= 32
  pl.hsum = pl.h + round256(rows * ffn * sizeof(uint16_t));
  pl.part = pl.hsum + round256(rows * (ffn / 32) * sizeof(float));
  pl.total = pl.part;
  pl.nsplit = 0;
  return pl;
}

static size_t prefill_split_bytes(int T, int k, int d) { return (size_t)T * k * d * sizeof(float); }

PrefillLayout prefill_layout(int T, int E, int k, int d, int ffn, int G) {
  const int tiles = prefill_tiles(T, E, k, d, ffn);
  PrefillLayout pl = prefill_layout_base(tiles, T, E, k, d, ffn);
  int s = prefill_nsplit(prefill_split(tiles, d, ffn, G), prefill_mt_planned(tiles, T, E, k));
  // a batch that fits the library's own scratch with fewer splits takes those
  const size_t split = prefill_split_bytes(T, k, d);
  if (pl.part + s * split > MC_NOALLOC_SCRATCH_BYTES && pl.part + split <= MC_NOALLOC_SCRATCH_BYTES)
    s = (int)((MC_NOALLOC_SCRATCH_BYTES - pl.part) / split);
  pl.nsplit = s;
  pl.total = pl.part + (size_t)s * split;
  return pl;
}

// The workspace query does not name the group size: the largest layout.
size_t prefill_workspace_bytes(int T, int E, int k, int d, int ffn) {
  return std::max({prefill_layout(T, E, k, d, ffn, 32).total, prefill_layout(T, E, k, d, ffn, 64).total,
                   prefill_layout(T, E, k, d, ffn, 128).total});
}

// The smallest T in (lo, hi] that satisfies f, hi if none before it does; f
// does not turn false again as T grows.
template <typename F>
static int first_T(int lo, int hi, F f) {
  while (hi - lo > 1) {
    const int mid = lo + (hi - lo) / 2;
    if (f(mid)) hi = mid;
    else lo = mid;
  }
  return hi;
}

// The largest prefill_workspace_bytes of the batches of lo to T tokens, without
// walking them all.  For one m-tile size and one number of splits the layout
// grows with T, so only the last T of each pair counts, and the splits repeat
// with the m-tile count's residue: at most `slots` counts back from the end of
// an m-tile size's range every number of splits has been met.  (The three
// layouts of every T up to 65536 took 14 ms.)  Batches that fit the scratch
// with one split need no more than it, however many they would take otherwise,
// and fewer bytes than one that does not fit.
size_t prefill_workspace_upto(int lo, int T, int E, int k, int d, int ffn) {
  const size_t scratch = MC_NOALLOC_SCRATCH_BYTES;
  const auto one_split = [&](int t) {
    return prefill_layout_base(prefill_tiles(t, E, k, d, ffn), t, E, k, d, ffn).total + prefill_split_bytes(t, k, d);
  };
  const bool in_scratch = one_split(T) <= scratch;
  if (!in_scratch && one_split(lo) <= scratch) lo = first_T(lo, T, [&](int t) { return one_split(t) > scratch; });
  size_t most = 0;
  for (int end = T; end >= lo;) {
    const int tiles = prefill_tiles(end, E, k, d, ffn);
    const auto same = [&](int t) { return prefill_tiles(t, E, k, d, ffn) >= tiles; };
    const int begin = same(lo) ? lo : first_T(lo, end, same);
    for (int G = 32; G <= 128; G *= 2) {
      const PrefillSplit sp = prefill_split(tiles, d, ffn, G);
      int met = 0;
      for (int t = end, n = 0; t >= begin && met < sp.most && n < sp.slots; ++n) {
        const long long mt = prefill_mt_planned(tiles, t, E, k);
        const int s = prefill_nsplit(sp, mt);
        if (s > met) {
          met = s;
          most = std::max(most, prefill_layout_base(tiles, t, E, k, d, ffn).total + s * prefill_split_bytes(t, k, d));
        }
        t = first_T(begin - 1, t, [&](int u) { return prefill_mt_planned(tiles, u, E, k) >= mt; }) - 1;
      }
    }
    end = begin - 1;
  }
  return in_scratch ? std::min(most, scratch) : most;
}

hipError_t launch_prefill(const uint16_t* x, const LayerArgs& L, const mc_routing& r, void* ws,
                          float** partial, size_t* part_stride, int* nsplit, hipStream_t stream,
                          const RouteArgs* route) {
  const PrefillLayout pl = prefill_layout(r.T, r.E, r.k, L.d, L.ffn, L.G);
  char* base = static_cast<char*>(ws);
  PrefillTables tb;
  int32_t* t = reinterpret_cast<int32_t*>(base + pl.tables);
  tb.ftile_base = t;
  tb.mt_e = t + (r.E + 1);
  tb.mt_j = tb.mt_e + pl.mt_max;
  tb.mt_count = tb.mt_j + pl.mt_max;
  tb.f_max = pl.f_max;
  tb.mt_max = pl.mt_max;
  tb.tiles = pl.tiles;
  tb.T = r.T;
  tb.P = r.T * r.k;
  uint16_t* xt = reinterpret_cast<uint16_t*>(base + pl.x);
  float* xsum = reinterpret_cast<float*>(base + pl.xsum);
  uint16_t* ht = reinterpret_cast<uint16_t*>(base + pl.h);
  float* hsum = reinterpret_cast<float*>(base + pl.hsum);
  *partial = reinterpret_cast<float*>(base + pl.part);
  *part_stride = (size_t)r.T * r.k * L.d;
  *nsplit = pl.nsplit;

  const dim3 pgrid(pl.f_max, (L.d + kGatherCols - 1) / kGatherCols);
  if (route) {
    timing_begin(stream, kSiteRouteFused);
#define MC_ROUTE_PREP(GP)                                                                                     \
  hipLaunchKernelGGL(route_prep_kernel<GP>, pgrid, dim3(64 * kRouteWaves), 0, stream, route->logits,          \
                     route->important, r.T, r.E, r.k, route->delta32, route->tau, route_bufs(r), x, L.d, tb, xt, xsum)
    if (L.G == 128) MC_ROUTE_PREP(16);
    else if (L.G == 64) MC_ROUTE_PREP(8);
    else MC_ROUTE_PREP(4);
#undef MC_ROUTE_PREP
    timing_end(stream, kSiteRouteFused);
  } else {
    timing_begin(stream, kSitePrefillPrep);
#define MC_PREP(GP)                                                                                           \
  hipLaunchKernelGGL(prefill_prep_kernel<GP>, pgrid, dim3(kGatherThreads), 0, stream, x, L.d, r.E, r.counts,  \
                     r.offsets, r.pair_token, tb, xt, xsum)
    if (L.G == 128) MC_PREP(16);
    else if (L.G == 64) MC_PREP(8);
    else MC_PREP(4);
#undef MC_PREP
    timing_end(stream, kSitePrefillPrep);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;

  PrefillGemm gu;
  gu.a = xt;
  gu.asum = xsum;
  gu.K = L.d;
  gu.n_tiles = L.ffn / prefill_rows(pl.tiles, L.G, true);
  gu.c_per_split = L.d / kTileCols;
  gu.nsplit = 1;
  gu.h = ht;
  gu.hsum = hsum;
  gu.partial = nullptr;
  gu.part_stride = 0;
  timing_begin(stream, kSiteGateUp);
  if (L.G == 128) err = launch_prefill_gemm<1>(L, r.offsets, tb, gu, true, pl.tiles, stream);
  else if (L.G == 64) err = launch_prefill_gemm<2>(L, r.offsets, tb, gu, true, pl.tiles, stream);
  else err = launch_prefill_gemm<4>(L, r.offsets, tb, gu, true, pl.tiles, stream);
  timing_end(stream, kSiteGateUp);
  if (err != hipSuccess) return err;

  PrefillGemm dn;
  const int ntk = L.ffn / kTileCols;
  dn.a = ht;
  dn.asum = hsum;
  dn.K = L.ffn;
  const int rows_dn = prefill_rows(pl.tiles, L.G, false);
  dn.n_tiles = (L.d + rows_dn - 1) / rows_dn;
  dn.c_per_split = (ntk + pl.nsplit - 1) / pl.nsplit;
  dn.nsplit = pl.nsplit;
  dn.h = nullptr;
  dn.hsum = nullptr;
  dn.partial = *partial;
  dn.part_stride = *part_stride;
  timing_begin(stream, kSiteDown);
  if (L.G == 128) err = launch_prefill_gemm<1>(L, r.offsets, tb, dn, false, pl.tiles, stream);
  else if (L.G == 64) err = launch_prefill_gemm<2>(L, r.offsets, tb, dn, false, pl.tiles, stream);
  else err = launch_prefill_gemm<4>(L, r.offsets, tb, dn, false, pl.tiles, stream);
  timing_end(stream, kSiteDown);
  return err;
}

}  // namespace mc
