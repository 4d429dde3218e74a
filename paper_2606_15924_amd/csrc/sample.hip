// Tile-wise error/age pixel sampling (Sec. 3.5).
//
// Three kernels per view:
//   tile_keys     eight lanes per tile (one thread with predicted weights): the
//                 integer tile weight (sum of E * 2^24) and the tile's race
//                 key, only when a subset of tiles is drawn;
//   tile_select   one workgroup: the tiles of the smallest race keys, listed
//                 ascending with their sample counts, prefix offsets and the
//                 tile -> slot map (every tile: a thread per tile, closed
//                 form);
//   tile_pixels   one wave per selected tile: N_hard sequential error-weighted
//                 draws without replacement, TopK age, uniform mixed draws.
// All decisions are integer: weights are exact integers (every finite
// non-negative half times 2^24 is one), a draw r = floor(u * W / 2^64) uses
// the high half of a 64 x 64-bit product, and the pick is the first pixel
// (ascending local index) whose running weight exceeds r.  Each lane owns four
// consecutive local indices, so lane order is index order and a wave prefix
// sum locates a draw.
//
// The tile pass draws tiles without replacement in proportion to weight.  Its
// order does not matter (tiles are listed ascending), so it runs as the
// exponential race of Efraimidis and Spirakis (IPL 2006), which has the
// sequential draws' distribution: tile t runs an Exp(1) time over its weight
// and the earliest n_sel win.  The time is exact integer and IEEE arithmetic:
// L = -log2 of the tile's uniform to 47 fractional bits (binary logarithm by
// repeated squaring), one correctly rounded double division L / w, and its bit
// pattern as the key; zero-weight tiles key 2^63 + u / 2, after every weighted
// tile.  Selection is an exact MSB-first radix select on the 64-bit keys, ties
// to the lower tile index.
#include <mutex>

#include "scan.h"

namespace tgs {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

// SplitMix64 finaliser (Steele, Lea & Flood 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t absorb(uint64_t h, uint64_t field) {
  return mix64(h + kGamma * (field + 1ull));
}

// Key of the (seed, step, view, tile) stream; a draw is absorb(key, slot).
__device__ __forceinline__ uint64_t stream_key(uint64_t seed, uint64_t step, uint64_t view,
                                               uint64_t tile) {
  return absorb(absorb(absorb(seed, step), view), tile);
}

__device__ __forceinline__ uint64_t mulhi64(uint64_t a, uint64_t b) { return __umul64hi(a, b); }

// E * 2^24 for a half bit pattern; negative, infinite and NaN values weigh 0.
__device__ __forceinline__ uint64_t half_weight(uint16_t h) {
  const uint32_t ex = (h >> 10) & 0x1f, man = h & 0x3ff;
  const uint64_t v = (uint64_t)(ex != 0 ? 1024u + man : man) << (max(ex, 1u) - 1u);  // no branch
  return h < 0x7c00 ? v : 0;
}

__device__ __forceinline__ int tile_valid_w(int tx, int W) { return min(kTile, W - tx * kTile); }
__device__ __forceinline__ int tile_valid_h(int ty, int H) { return min(kTile, H - ty * kTile); }

// ------------------------------------------------------------------ arguments
// A view's arguments; the views of a step share the launches, one per grid
// layer.
struct SampleArgs {
  const uint16_t* E;
  const uint16_t* A;
  const float* pred;  // nullable
  uint64_t* keys;
  int32_t* valid_tiles;
  int32_t* tile_off;
  int32_t* tile_slot;
  uint8_t* pix;
  int H, W, tiles_x, tiles_y;
  int n_st;
  uint64_t view;
};

// What the views share.
struct SampleCommon {
  int n_sel, n_pix, hard_pm, stable_pm;
  uint64_t seed, step;
  int64_t* totals;
};

// ------------------------------------------------------------------ race keys
constexpr int kLogFrac = 47;  // fractional bits of a race time: 64 * 2^47 = 2^53 is exact in a double

// 2^47 * -log2(v / 2^64) for v = u | 1, the fraction truncated: with
// v = 2^e m, m in [1, 2), the time is 64 - e - log2(m), and each squaring of m
// (held in Q1.63, truncated) yields the next bit of log2(m): bit 1 and
// m <- m^2 / 2 when m^2 >= 2, else bit 0 and m <- m^2.
__device__ __forceinline__ uint64_t neg_log2_fixed(uint64_t u) {
  const uint64_t v = u | 1ull;
  const int e = 63 - __clzll((long long)v);
  uint64_t m = v << (63 - e);
  uint64_t frac = 0;
#pragma unroll 4
  for (int k = 0; k < kLogFrac; ++k) {
    const uint64_t hi = __umul64hi(m, m);
    const uint64_t lo_top = (m * m) >> 63;
    const uint64_t bit = hi >> 63;
    frac = (frac << 1) | bit;
    m = bit ? hi : ((hi << 1) | lo_top);
  }
  return ((uint64_t)(64 - e) << kLogFrac) - frac;
}

// Race key of a tile of weight w whose uniform is u: the bit pattern of the
// positive double L / w (ordered like the doubles, below 2^63), or 2^63 + u / 2
// for w = 0.
__device__ __forceinline__ uint64_t race_key(uint64_t w, uint64_t u) {
  if (w == 0) return (1ull << 63) | (u >> 1);
  return (uint64_t)__double_as_longlong(__ddiv_rn((double)neg_log2_fixed(u), (double)w));
}

// Eight tiles per wave, eight lanes per tile: lane k of a tile's group sums
// its pixels k, k + 8, ... (32 of them, a half row per load across the
// group), a butterfly over the group adds the eight 64-bit partial sums
// exactly, and the group's first lane computes the key, eight keys in
// parallel per wave.
constexpr int kKeyTiles = 8;

__global__ void __launch_bounds__(64) tile_keys_kernel(Batch<SampleArgs> batch, SampleCommon c) {
  const SampleArgs& v = batch.v[blockIdx.z];
  const uint16_t* __restrict__ const E = v.E;
  const int H = v.H, W = v.W, tiles_x = v.tiles_x, n_t = v.tiles_x * v.tiles_y;
  const int lane = threadIdx.x;
  const int sub = lane & (kKeyTiles - 1);
  const int t = blockIdx.x * kKeyTiles + lane / kKeyTiles;
  uint64_t s = 0;
  if (t < n_t) {
    const int tx = t % tiles_x, ty = t / tiles_x;
#pragma unroll 8
    for (int k = 0; k < kTilePixels / kKeyTiles; ++k) {
      const int loc = sub + kKeyTiles * k;
      const int x = tx * kTile + (loc & 15), y = ty * kTile + (loc >> 4);
      // a clamped address, so that no load waits behind a branch
      const uint64_t w = half_weight(E[(int64_t)min(y, H - 1) * W + min(x, W - 1)]);
      s += x < W && y < H ? w : 0;
    }
  }
#pragma unroll
  for (int o = 1; o < kKeyTiles; o <<= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)s, o, kWave);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(s >> 32), o, kWave);
    s += ((uint64_t)hi << 32) | lo;
  }
  if (t < n_t && sub == 0)
    v.keys[t] = race_key(s, absorb(stream_key(c.seed, c.step, v.view, (uint64_t)n_t), (uint64_t)t));
}

// Keys from predicted mean tile errors: weight floor(clamp(p, 0, 65504) *
// in-image pixels * 2^24), the units of the error-map sums; exact in FP64 (a
// float times a count up to 256 times a power of two).
__global__ void __launch_bounds__(256) tile_pred_keys_kernel(Batch<SampleArgs> batch, SampleCommon c) {
  const SampleArgs& v = batch.v[blockIdx.z];
  const int H = v.H, W = v.W, tiles_x = v.tiles_x, n_t = v.tiles_x * v.tiles_y;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n_t) return;
  const int tx = t % tiles_x, ty = t / tiles_x;
  const int nx = min(kTile, W - tx * kTile), ny = min(kTile, H - ty * kTile);
  const float p = v.pred[t];
  const double q = p > 0.f ? (double)fminf(p, 65504.f) : 0.0;  // NaN and negatives give 0
  const uint64_t w = (uint64_t)floor(q * (double)(nx * ny) * 16777216.0);
  v.keys[t] = race_key(w, absorb(stream_key(c.seed, c.step, v.view, (uint64_t)n_t), (uint64_t)t));
}

// ------------------------------------------------------------------ tile select
// Every tile: a thread per tile writes its slot and its sample offset in
// closed form (every tile column but the last is 16 pixels wide, every row
// but the last 16 high), so no single-workgroup pass has to wait for a free
// compute unit while other streams' kernels fill the device.
__global__ void __launch_bounds__(256) tile_list_all_kernel(Batch<SampleArgs> batch, SampleCommon c) {
  const SampleArgs& v = batch.v[blockIdx.z];
  const int H = v.H, W = v.W, tiles_x = v.tiles_x, tiles_y = v.tiles_y, n_pix = c.n_pix;
  const int n_t = tiles_x * tiles_y;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t > n_t) return;
  const int wl = W - (tiles_x - 1) * kTile, hl = H - (tiles_y - 1) * kTile;  // last column's width, last row's height
  const int64_t row16 = (int64_t)(tiles_x - 1) * min(n_pix, kTile * kTile) + min(n_pix, wl * kTile);
  const int ty = t / tiles_x, tx = t % tiles_x;  // t = n_t: ty = tiles_y, tx = 0
  int64_t off = (int64_t)min(ty, tiles_y - 1) * row16;
  if (ty == tiles_y) off += (int64_t)(tiles_x - 1) * min(n_pix, kTile * hl) + min(n_pix, wl * hl);
  else off += (int64_t)tx * min(n_pix, kTile * (ty == tiles_y - 1 ? hl : kTile));
  v.tile_off[t] = (int32_t)off;
  if (t < n_t) {
    v.valid_tiles[t] = t;
    v.tile_slot[t] = t;
  } else {
    atomicAdd((unsigned long long*)&c.totals[0], (unsigned long long)off);
    atomicAdd((unsigned long long*)&c.totals[1], (unsigned long long)n_t);
  }
}

// A subset: one workgroup.  A radix select over the race keys (11 bits a
// pass from the highest bit in which any two keys differ, LDS histogram)
// narrows the n_sel-th smallest key down to a few candidates, which are
// ranked against each other; thr is that key and krem how many of the keys
// equal to it are taken (the lowest tile indices first).  Then the whole
// workgroup lists the chosen tiles in ascending order with their sample
// counts and prefix offsets, a tile per thread and round.
//
// Bound by the instructions that one compute unit issues and by barriers, so
// the keys stay in registers (kRegs: all rounds at once; a grid of more
// tiles than the largest such variant reads them again from memory in each
// pass), and a grid of few tiles takes a small workgroup: 8,160 tiles 13 us,
// 256 tiles 5.5 us.  With the keys in LDS, 8-bit passes from bit 63 on and a
// contiguous run of tiles per thread in the listing: 25 and 7 us; the same
// 11-bit passes with keys in LDS and 1024 threads throughout: 23 and 11 us.
constexpr int kSelectBits = 11;
constexpr int kSelectBins = 1 << kSelectBits;
constexpr int kRankCandidates = 128;

__device__ __forceinline__ uint64_t wave_or_u64(uint64_t v) {
  uint32_t w[2] = {(uint32_t)v, (uint32_t)(v >> 32)};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    int x = (int)w[k];
    x |= dpp_i<kDppQuadPerm1032>(0, x);
    x |= dpp_i<kDppQuadPerm2301>(0, x);
    x |= dpp_i<kDppRowHalfMirror>(0, x);
    x |= dpp_i<kDppRowMirror>(0, x);
    x |= dpp_i<kDppRowBcast15, 0xa>(0, x);
    x |= dpp_i<kDppRowBcast31, 0xc>(0, x);
    w[k] = (uint32_t)__builtin_amdgcn_readlane(x, 63);
  }
  return (uint64_t)w[1] << 32 | w[0];
}

// Exclusive prefix over the workgroup of a value per thread (in lds, kThreads
// / 64 entries), the sum in *total.  Barriers before and after lds is used.
template <int kThreads>
__device__ __forceinline__ uint64_t select_scan(uint64_t v, uint64_t* lds, uint64_t* total) {
  constexpr int kWaves = kThreads / kWave;
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  const uint64_t incl = wave_inclusive_scan_u64_dpp(v);
  if (lane == kWave - 1) lds[wave] = incl;
  __syncthreads();
  const uint64_t w = lane < kWaves ? lds[lane] : 0;
  const uint64_t wi = wave_inclusive_scan_u64_dpp(w);
  *total = readlane_u64(wi, kWaves - 1);
  const uint64_t before = readlane_u64(wi - w, __builtin_amdgcn_readfirstlane(wave));
  __syncthreads();
  return before + incl - v;
}

template <int kThreads, int kItems, bool kRegs>
__global__ void __launch_bounds__(kThreads) tile_select_kernel(Batch<SampleArgs> batch, SampleCommon common) {
  const SampleArgs& v = batch.v[blockIdx.z];
  const uint64_t* __restrict__ const keys = v.keys;
  int32_t* __restrict__ const valid_tiles = v.valid_tiles;
  int32_t* __restrict__ const tile_off = v.tile_off;
  int32_t* __restrict__ const tile_slot = v.tile_slot;
  int64_t* __restrict__ const totals = common.totals;
  const int H = v.H, W = v.W, tiles_x = v.tiles_x, tiles_y = v.tiles_y, n_sel = common.n_sel, n_pix = common.n_pix;
  constexpr int kWaves = kThreads / kWave;
  constexpr int kStep = kThreads * kItems;
  static_assert(kItems * kWaves <= kThreads && kItems <= 32, "a count per wave and round");
  __shared__ uint32_t hist[kSelectBins];
  __shared__ uint64_t lds[kWaves], s_or[2 * kWaves];
  __shared__ uint64_t s_n[kItems * kWaves];  // tiles above, samples below bit 32
  __shared__ uint64_t s_cand[kRankCandidates];
  __shared__ uint64_t s_thr;
  __shared__ int s_krem, s_in_bin, s_cands;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int n_t = tiles_x * tiles_y;  // 0 <= n_sel < n_t; at most kStep when kRegs
  uint64_t k[kItems];
  auto load = [&](int t0) {
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int t = t0 + i * kThreads + tid;
      k[i] = keys[min(t, n_t - 1)];
    }
  };
  auto is_tile = [&](int t0, int i) { return t0 + i * kThreads + tid < n_t; };
  if (kRegs) load(0);
  uint64_t thr = 0;
  int krem = 0;
  int fs = 0;             // keys are compared on their bits from fs up
  bool all_ties = false;  // every key equal to thr on those bits is chosen
  if (n_sel > 0) {
    // the bits in which the keys differ: set in some key and clear in another
    uint64_t any = 0, none = 0;
    for (int t0 = 0; t0 < n_t; t0 += kStep) {
      if (!kRegs) load(t0);
#pragma unroll
      for (int i = 0; i < kItems; ++i) {  // past the end: the last tile's key again
        any |= k[i];
        none |= ~k[i];
      }
    }
    any = wave_or_u64(any);
    none = wave_or_u64(none);
    if (lane == 0) {
      s_or[wave] = any;
      s_or[kWaves + wave] = none;
    }
    if (tid == 0) s_cands = 0;
    __syncthreads();
    any = wave_or_u64(lane < kWaves ? s_or[lane] : 0);
    none = wave_or_u64(lane < kWaves ? s_or[kWaves + lane] : 0);
    const uint64_t differ = any & none;
    int top = differ != 0 ? 64 - __clzll((long long)differ) : 0;  // bits still open: [0, top)
    thr = any & ~(top < 64 ? (1ull << top) - 1 : ~0ull);          // the bits above, which every key shares
    krem = n_sel;
    int in_bin = n_t;  // keys that share thr's bits from top up
    while (top > 0 && in_bin != krem && in_bin > kRankCandidates) {
      const int shift = max(top - kSelectBits, 0);
      const uint32_t dmask = (1u << (top - shift)) - 1u;
      for (int b = tid; b < kSelectBins; b += kThreads) hist[b] = 0;
      __syncthreads();
      const uint64_t hmask = top == 64 ? 0ull : ~0ull << top;  // bits already fixed
      for (int t0 = 0; t0 < n_t; t0 += kStep) {
        if (!kRegs) load(t0);
#pragma unroll
        for (int i = 0; i < kItems; ++i)
          if (is_tile(t0, i) && ((k[i] ^ thr) & hmask) == 0) atomicAdd(&hist[(uint32_t)(k[i] >> shift) & dmask], 1u);
      }
      __syncthreads();
      // the bin in which the running count reaches krem (the candidates
      // number at least krem)
      constexpr int kBins = kSelectBins / kThreads;
      uint32_t h[kBins], sum = 0;
#pragma unroll
      for (int i = 0; i < kBins; ++i) {
        h[i] = hist[tid * kBins + i];
        sum += h[i];
      }
      uint64_t all;
      uint32_t below = (uint32_t)select_scan<kThreads>(sum, lds, &all);
#pragma unroll
      for (int i = 0; i < kBins; ++i) {
        if (below < (uint32_t)krem && below + h[i] >= (uint32_t)krem) {
          s_thr = thr | ((uint64_t)(tid * kBins + i) << shift);
          s_krem = krem - (int)below;
          s_in_bin = (int)h[i];
        }
        below += h[i];
      }
      __syncthreads();
      thr = s_thr;
      krem = s_krem;
      in_bin = s_in_bin;
      top = shift;
    }
    fs = top;
    if (in_bin == krem) {
      all_ties = true;  // every key with this prefix is chosen: the lower bits decide nothing
    } else if (top > 0) {
      // few candidates: the one with fewer than krem below it and krem or
      // more up to and with it is thr
      const uint64_t hmask = top == 64 ? 0ull : ~0ull << top;
      for (int t0 = 0; t0 < n_t; t0 += kStep) {
        if (!kRegs) load(t0);
#pragma unroll
        for (int i = 0; i < kItems; ++i)
          if (is_tile(t0, i) && ((k[i] ^ thr) & hmask) == 0) {
            const int at = atomicAdd(&s_cands, 1);
            if (at < kRankCandidates) s_cand[at] = k[i];  // always: in_bin candidates
          }
      }
      __syncthreads();
      const int cands = min(s_cands, kRankCandidates);
      if (tid < cands) {
        const uint64_t mine = s_cand[tid];
        int less = 0, equal = 0;
#pragma unroll 4
        for (int c = 0; c < cands; ++c) {
          less += s_cand[c] < mine ? 1 : 0;
          equal += s_cand[c] == mine ? 1 : 0;
        }
        if (less < krem && less + equal >= krem) {  // equal keys write the same
          s_thr = mine;
          s_krem = krem - less;
          s_in_bin = equal;
        }
      }
      __syncthreads();
      thr = s_thr;
      krem = s_krem;
      all_ties = s_in_bin == krem;
      fs = 0;
    }
  }
  // the list of the chosen tiles: keys below thr, and the first krem tiles
  // whose key equals thr, both on the bits from fs up.  One count per wave
  // and round, scanned together.  A tile has pf samples, fewer in the last
  // column (dc more, negative) and the last row (dr); the corner (both) is
  // the last tile, and its own difference dk is in no other tile's offset.
  const uint64_t thr_s = thr >> fs;
  const int w0 = tiles_x > 1 ? kTile : W, h0 = tiles_y > 1 ? kTile : H;
  const int w1 = tile_valid_w(tiles_x - 1, W), h1 = tile_valid_h(tiles_y - 1, H);
  const int pf = min(n_pix, w0 * h0), dc = min(n_pix, w1 * h0) - pf, dr = min(n_pix, w0 * h1) - pf;
  const int dk = min(n_pix, w1 * h1) - pf - dc - dr;
  const bool ragged = (dc | dr | dk) != 0;
  // exclusive prefixes of s_n; returns the sum
  auto scan_counts = [&] {
    __syncthreads();
    uint64_t all;
    const uint64_t ex = select_scan<kThreads>(tid < kItems * kWaves ? s_n[tid] : 0ull, lds, &all);
    if (tid < kItems * kWaves) s_n[tid] = ex;
    __syncthreads();
    return all;
  };
  uint32_t ties_before = 0;
  uint64_t done = 0;  // as s_n
  for (int t0 = 0; t0 < n_t; t0 += kStep) {
    if (!kRegs) load(t0);
    uint32_t chosen = 0, tied = 0;  // bit i: this thread's tile of round i
    if (n_sel > 0) {
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        const uint64_t ks = k[i] >> fs;
        if (is_tile(t0, i) && ks < thr_s) chosen |= 1u << i;
        if (is_tile(t0, i) && ks == thr_s) tied |= 1u << i;
      }
      if (all_ties) {
        chosen |= tied;
      } else {  // equal 64-bit keys, not all of them taken
        for (int i = 0; i < kItems; ++i) {
          const uint64_t m = ballot((tied >> i) & 1u);
          if (lane == 0) s_n[i * kWaves + wave] = (uint64_t)__popcll(m);
        }
        const uint64_t all = scan_counts();
        for (int i = 0; i < kItems; ++i) {
          const bool tie = (tied >> i) & 1u;
          const uint64_t m = ballot(tie);
          const uint32_t rank = ties_before + (uint32_t)s_n[i * kWaves + wave] + (uint32_t)mask_rank(m);
          if (tie && rank < (uint32_t)krem) chosen |= 1u << i;
        }
        ties_before += (uint32_t)all;
        __syncthreads();  // s_n is written again below
      }
    }
    uint32_t last_col = 0, last_row = 0;  // bits as chosen, of the chosen tiles
    if (ragged) {
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        const int t = t0 + i * kThreads + tid;
        if ((t + 1) % tiles_x == 0) last_col |= 1u << i;
        if (t >= n_t - tiles_x) last_row |= 1u << i;
      }
      last_col &= chosen;
      last_row &= chosen;
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int n = __popcll(ballot((chosen >> i) & 1u));
      int p = n * pf;
      if (ragged) {
        const uint64_t mc = ballot((last_col >> i) & 1u), mr = ballot((last_row >> i) & 1u);
        const bool corner = ballot(((chosen >> i) & 1u) && t0 + i * kThreads + tid == n_t - 1) != 0;
        p += __popcll(mc) * dc + __popcll(mr) * dr + (corner ? dk : 0);
      }
      if (lane == 0) s_n[i * kWaves + wave] = (uint64_t)n << 32 | (uint32_t)p;
    }
    const uint64_t all = scan_counts();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int t = t0 + i * kThreads + tid;
      const bool ch = (chosen >> i) & 1u;
      const int rank = mask_rank(ballot(ch));
      int p = rank * pf;
      if (ragged)
        p += mask_rank(ballot((last_col >> i) & 1u)) * dc + mask_rank(ballot((last_row >> i) & 1u)) * dr;
      const uint64_t before = done + s_n[i * kWaves + wave];
      const int slot = ch ? (int)(before >> 32) + rank : -1;
      if (t >= n_t) continue;
      if (ch) {
        valid_tiles[slot] = t;
        tile_off[slot] = (int32_t)(uint32_t)before + p;
      }
      tile_slot[t] = slot;
    }
    done += all;
    if (!kRegs) __syncthreads();
  }
  if (tid == 0) {
    tile_off[done >> 32] = (int32_t)(uint32_t)done;
    atomicAdd((unsigned long long*)&totals[0], (unsigned long long)(uint32_t)done);
    atomicAdd((unsigned long long*)&totals[1], (unsigned long long)(done >> 32));
  }
}

// ------------------------------------------------------------------ tile pixels
__device__ __forceinline__ int split_round(int permille, int n) { return (permille * n + 500) / 1000; }

// One wave per tile.  Bound by the chain of draws (each needs the weight that
// the last one left) of the few waves that a view gives a SIMD: the draws
// update running sums without a branch, the counts are ballots, the loads
// wait for nothing.  4,293 tiles of 64 samples (1296x840): 23 us; with the
// in-lane search in a branch, 24 counting steps by lane sums for the ages and
// loads behind the image bounds it took 47 us.  6,120 tiles of 51: 21 us.
__global__ void __launch_bounds__(64) tile_pixels_kernel(Batch<SampleArgs> batch, SampleCommon common) {
  const SampleArgs& v = batch.v[blockIdx.z];
  const uint16_t* __restrict__ const E = v.E;
  const uint16_t* __restrict__ const A = v.A;
  const int32_t* __restrict__ const valid_tiles = v.valid_tiles;
  const int32_t* __restrict__ const tile_off = v.tile_off;
  uint8_t* __restrict__ const pix = v.pix;
  const int H = v.H, W = v.W, tiles_x = v.tiles_x, n_st = v.n_st, n_pix = common.n_pix;
  const int hard_pm = common.hard_pm, stable_pm = common.stable_pm;
  const int slot = blockIdx.x;
  if (slot >= n_st) return;
  const int lane = threadIdx.x;
  const int t = valid_tiles[slot], out = tile_off[slot];
  const int tx = t % tiles_x, ty = t / tiles_x;
  const int n_valid = tile_valid_w(tx, W) * tile_valid_h(ty, H);
  const int n = min(n_pix, n_valid);
  int n_hard = split_round(hard_pm, n);
  int n_stable = split_round(stable_pm, n);
  if (n_hard + n_stable > n) n_stable = n - n_hard;
  int n_mixed = n - n_hard - n_stable;

  // The lane's four pixels are consecutive in a row.  Out-of-image pixels
  // load a clamped address, so that no load waits behind a branch.
  uint64_t w[4];
  int age[4];
  bool valid[4];
  {
    const int x0 = tx * kTile + (lane & 3) * 4, y = ty * kTile + (lane >> 2);
    const int64_t row = (int64_t)min(y, H - 1) * W;
    uint16_t e[4], g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t idx = row + min(x0 + k, W - 1);
      e[k] = E[idx];
      g[k] = A[idx];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      valid[k] = x0 + k < W && y < H;
      w[k] = valid[k] ? half_weight(e[k]) : 0;
      age[k] = g[k];
    }
  }
  uint32_t picked = 0;  // bit k: local index lane*4+k chosen
  const uint64_t key = stream_key(common.seed, common.step, v.view, (uint64_t)t);

  // --- hard: sequential error-weighted draws without replacement.  The
  // draws' random words are hashed up front, lane l holding draw l + 64 q
  // in uh[q].  c[k] is the running weight, over the whole tile, up to and
  // with pixel k: a draw r picks the first pixel with c > r, and taking its
  // weight away lowers exactly the sums that exceed r.  A picked pixel's sum
  // then equals its predecessor's, so it is never the first above a draw
  // again, and after the draws the pixels of positive weight whose sum
  // equals their predecessor's are the picked ones.
  int n_hard_done = 0;
  {
    uint64_t uh[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) uh[q] = kWave * q < n_hard ? absorb(key, (uint64_t)(lane + kWave * q)) : 0;
    const uint64_t ls = w[0] + w[1] + w[2] + w[3];
    uint64_t c[4];
    c[3] = wave_inclusive_scan_u64_dpp(ls);
    c[2] = c[3] - w[3];
    c[1] = c[2] - w[2];
    c[0] = c[1] - w[1];
    uint64_t total = readlane_u64(c[3], kWave - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      for (int jj = 0; jj < kWave && n_hard_done < n_hard && total != 0; ++jj) {
        const uint64_t r = mulhi64(readlane_u64(uh[q], jj), total);
        const bool above0 = c[0] > r, above1 = c[1] > r, above2 = c[2] > r, above3 = c[3] > r;
        const int pl = (int)__builtin_ctzll(ballot(above3));  // c[3] of lane 63 = total > r
        const uint64_t wp = readlane_u64(above0 ? w[0] : above1 ? w[1] : above2 ? w[2] : w[3], pl);
        c[0] -= above0 ? wp : 0;
        c[1] -= above1 ? wp : 0;
        c[2] -= above2 ? wp : 0;
        c[3] -= above3 ? wp : 0;
        total -= wp;
        ++n_hard_done;
      }
    }
    const uint32_t plo = (uint32_t)__shfl_up((int)(uint32_t)c[3], 1, kWave);
    const uint32_t phi = (uint32_t)__shfl_up((int)(uint32_t)(c[3] >> 32), 1, kWave);
    uint64_t prev = lane == 0 ? 0 : ((uint64_t)phi << 32) | plo;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (w[k] != 0 && c[k] == prev) picked |= 1u << k;
      prev = c[k];
    }
  }
  n_mixed += n_hard - n_hard_done;

  // --- stable: TopK age among the rest, ties to the lower index.  The K-th
  // largest age is built bit by bit on counts.
  if (n_stable > 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (!valid[k] || ((picked >> k) & 1u)) age[k] = -1;
    auto count = [&](int a) {  // pixels of at least age a
      int c = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) c += __builtin_popcountll(ballot(age[k] >= a));
      return c;
    };
    int kth = 0;
    for (int bit = count(256) >= n_stable ? 1 << 15 : 1 << 7; bit > 0; bit >>= 1)
      if (count(kth | bit) >= n_stable) kth |= bit;
    const int ties = n_stable - count(kth + 1);  // to take among those of the K-th age
    int lt = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) lt += age[k] == kth ? 1 : 0;
    int before = wave_inclusive_scan_i_dpp(lt) - lt;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (age[k] > kth || (age[k] == kth && before++ < ties)) picked |= 1u << k;
  }

  // --- mixed: uniform without replacement over the rest: a draw picks the
  // r-th remaining pixel in ascending order.  c[k] counts the remaining
  // pixels up to and with pixel k and is kept up to date as above; each draw
  // takes one pixel, so every r is known up front.
  {
    int c[4], lc = 0;
    bool rest[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      rest[k] = valid[k] && !((picked >> k) & 1u);
      lc += rest[k] ? 1 : 0;
    }
    c[3] = wave_inclusive_scan_i_dpp(lc);
    c[2] = c[3] - (rest[3] ? 1 : 0);
    c[1] = c[2] - (rest[2] ? 1 : 0);
    c[0] = c[1] - (rest[1] ? 1 : 0);
    const int nrem = __builtin_amdgcn_readlane(c[3], kWave - 1);
    const int draws = min(n_mixed, nrem);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (kWave * q >= draws) continue;  // uniform
      const int j = lane + kWave * q;
      const int rj = (int)mulhi64(absorb(key, (uint64_t)(256 + j)), (uint64_t)max(nrem - j, 0));
      for (int jj = 0; jj < min(kWave, draws - kWave * q); ++jj) {
        const int r = __builtin_amdgcn_readlane(rj, jj);
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] -= c[k] > r ? 1 : 0;
      }
    }
    int prev = __shfl_up(c[3], 1, kWave);
    if (lane == 0) prev = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (rest[k] && c[k] == prev) picked |= 1u << k;
      prev = c[k];
    }
  }

  // --- write the sorted local indices
  const int lc = __builtin_popcount(picked);
  const int ic = wave_inclusive_scan_i_dpp(lc);
  int pos = out + ic - lc;
  for (int k = 0; k < 4; ++k)
    if ((picked >> k) & 1u) pix[pos++] = (uint8_t)(lane * 4 + k);
}

}  // namespace tgs

using namespace tgs;

extern "C" size_t tgs_sample_workspace_size(int32_t height, int32_t width) {
  if (height <= 0 || width <= 0) return 0;
  const size_t n_t = (size_t)(ceil_div(width, kTile) * ceil_div(height, kTile));
  return align_up(n_t * sizeof(uint64_t), 256);
}

static int32_t sample_args(SampleArgs& v, const uint16_t* E, const uint16_t* A, int32_t height, int32_t width,
                           const tgs_sample_params* sp, int32_t view, const float* tile_pred, int32_t* valid_tiles,
                           int32_t* tile_off, uint8_t* pix, int32_t* tile_slot, const int64_t* totals, void* ws,
                           size_t ws_bytes) {
  TGS_REQUIRE(height > 0 && width > 0, "tgs_sample: bad image size %d x %d", width, height);
  TGS_REQUIRE(sp != nullptr, "tgs_sample: null params");
  TGS_REQUIRE(sp->n_pix >= 1 && sp->n_pix <= kTilePixels, "tgs_sample: n_pix %d not in 1..256",
              sp->n_pix);
  TGS_REQUIRE(sp->hard_permille >= 0 && sp->stable_permille >= 0 &&
                  sp->hard_permille + sp->stable_permille <= 1000,
              "tgs_sample: bad hard/stable ratios");
  TGS_REQUIRE(view >= 0, "tgs_sample: negative view index");
  TGS_REQUIRE(E && A && valid_tiles && tile_off && pix && tile_slot && totals && ws,
              "tgs_sample: null pointer");
  TGS_REQUIRE(ws_bytes >= tgs_sample_workspace_size(height, width),
              "tgs_sample: workspace %zu bytes < %zu", ws_bytes,
              tgs_sample_workspace_size(height, width));
  v = SampleArgs{E,    A,      tile_pred, (uint64_t*)ws, valid_tiles, tile_off, tile_slot, pix, height, width,
                 (int)ceil_div(width, kTile), (int)ceil_div(height, kTile), tgs_sample_tile_count(height, width, sp),
                 (uint64_t)view};
  return TGS_OK;
}

static bool all_tiles(const SampleArgs& v, const tgs_sample_params* sp) {
  return sp->n_tiles_sel < 0 || sp->n_tiles_sel >= v.tiles_x * v.tiles_y;
}

// Views whose tiles are drawn the same way: all of them, by the error map or
// by the predictions.
static void sample_launch(const Batch<SampleArgs>& b, int views, const tgs_sample_params* sp, int64_t* totals,
                          hipStream_t s) {
  const SampleCommon c{sp->n_tiles_sel, sp->n_pix, sp->hard_permille, sp->stable_permille, sp->seed, sp->step, totals};
  const unsigned nv = (unsigned)views;
  int n_t = 0, n_st = 0;
  for (int k = 0; k < views; ++k) {
    n_t = max(n_t, b.v[k].tiles_x * b.v[k].tiles_y);
    n_st = max(n_st, b.v[k].n_st);
  }
  if (all_tiles(b.v[0], sp)) {
    hipLaunchKernelGGL(tile_list_all_kernel, dim3((unsigned)ceil_div(n_t + 1, 256), 1, nv), dim3(256), 0, s, b, c);
  } else {
    if (b.v[0].pred != nullptr)
      hipLaunchKernelGGL(tile_pred_keys_kernel, dim3((unsigned)ceil_div(n_t, 256), 1, nv), dim3(256), 0, s, b, c);
    else
      hipLaunchKernelGGL(tile_keys_kernel, dim3((unsigned)ceil_div(n_t, kKeyTiles), 1, nv), dim3(64), 0, s, b, c);
    auto select = [&](auto kernel, int threads) {
      hipLaunchKernelGGL(kernel, dim3(1, 1, nv), dim3(threads), 0, s, b, c);
    };
    // the smallest variant that keeps every key in registers
    if (n_t <= 256 * 4) select(tile_select_kernel<256, 4, true>, 256);
    else if (n_t <= 1024 * 8) select(tile_select_kernel<1024, 8, true>, 1024);
    else if (n_t <= 1024 * 16) select(tile_select_kernel<1024, 16, true>, 1024);
    else select(tile_select_kernel<1024, 16, false>, 1024);
  }
  if (n_st > 0)
    hipLaunchKernelGGL(tile_pixels_kernel, dim3((unsigned)n_st, 1, nv), dim3(64), 0, s, b, c);
}

static int32_t sample_impl(const uint16_t* E, const uint16_t* A, int32_t height, int32_t width,
                           const tgs_sample_params* sp, const float* tile_pred, int32_t* valid_tiles,
                           int32_t* tile_off, uint8_t* pix, int32_t* tile_slot, int64_t* totals, void* ws,
                           size_t ws_bytes, void* stream) {
  Batch<SampleArgs> b{};
  if (int32_t e = sample_args(b.v[0], E, A, height, width, sp, sp != nullptr ? sp->view : 0, tile_pred, valid_tiles,
                              tile_off, pix, tile_slot, totals, ws, ws_bytes))
    return e;
  sample_launch(b, 1, sp, totals, as_stream(stream));
  return hip_status("tgs_sample");
}

extern "C" int32_t tgs_sample_views(const tgs_view* views, int32_t n_views, const tgs_sample_params* sp,
                                    int64_t* totals, void* stream) {
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || views != nullptr), "tgs_sample_views: bad view list");
  for (int pass = 0; pass < 2; ++pass)  // every view is checked before any is launched
    for (int32_t k = 0, end; k < n_views; k = end) {
      Batch<SampleArgs> b{};
      for (end = k; end < n_views && end - k < kBatch; ++end) {
        const tgs_view& v = views[end];
        SampleArgs a{};
        if (int32_t e = sample_args(a, v.E, v.A, v.height, v.width, sp, v.view, v.tile_pred, v.valid_tiles, v.tile_off,
                                    v.pix, v.tile_slot, totals, v.sample_ws, v.sample_ws_bytes))
          return e;
        if (end > k && (all_tiles(a, sp) != all_tiles(b.v[0], sp) || (a.pred == nullptr) != (b.v[0].pred == nullptr)))
          break;
        b.v[end - k] = a;
      }
      if (pass == 1) sample_launch(b, end - k, sp, totals, as_stream(stream));
    }
  return hip_status("tgs_sample_views");
}

extern "C" int32_t tgs_sample(const uint16_t* E, const uint16_t* A, int32_t height, int32_t width,
                              const tgs_sample_params* sp, const float* tile_pred, int32_t* valid_tiles,
                              int32_t* tile_off, uint8_t* pix, int32_t* tile_slot, int64_t* totals, void* ws,
                              size_t ws_bytes, void* stream) {
  return sample_impl(E, A, height, width, sp, tile_pred, valid_tiles, tile_off, pix, tile_slot, totals, ws,
                     ws_bytes, stream);
}

// ------------------------------------------------------------------ sampling without a workspace
// The sampler's scratch (the tiles' race keys, 8 bytes per tile)
// in a file-scope device array, for callers that cannot allocate.  Each
// GPU holds its own copy until the process ends; host code uses only the
// device address that hipGetSymbolAddress returns for the current device,
// never the array's name.  Every kernel of a call writes the scratch it
// reads, so nothing needs clearing between calls; calls that overlap on
// one GPU share it and race.
constexpr int kNoAllocMaxTiles = TGS_SAMPLE_NOALLOC_MAX_TILES;
constexpr size_t kNoAllocScratchBytes =
    ((size_t)kNoAllocMaxTiles * sizeof(uint64_t) + 255) / 256 * 256;
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

// The current device's address of the scratch array, looked up on the
// first call on that device.
static void* scratch_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

extern "C" int32_t tgs_sample_noalloc(const uint16_t* E, const uint16_t* A, int32_t height, int32_t width,
                                      const tgs_sample_params* sp, const float* tile_pred, int32_t* valid_tiles,
                                      int32_t* tile_off, uint8_t* pix, int32_t* tile_slot, int64_t* totals,
                                      void* stream) {
  TGS_REQUIRE(height > 0 && width > 0, "tgs_sample_noalloc: bad image size %d x %d", width, height);
  const int64_t n_t = ceil_div(width, kTile) * ceil_div(height, kTile);
  TGS_REQUIRE(n_t <= kNoAllocMaxTiles, "tgs_sample_noalloc: %lld tiles exceed the static scratch of %d tiles",
              (long long)n_t, kNoAllocMaxTiles);
  void* ws = scratch_address();
  if (ws == nullptr) {
    set_error("tgs_sample_noalloc: no device address for the static scratch");
    return TGS_ERR_HIP;
  }
  return sample_impl(E, A, height, width, sp, tile_pred, valid_tiles, tile_off, pix, tile_slot, totals, ws,
                     kNoAllocScratchBytes, stream);
}

// ------------------------------------------------------------------ per-view mean error
// Eq. anchor_view needs each view's mean error E_bar_v over the image: the
// exact integer sum of the half values times 2^24 (the weights above), one
// 64-bit atomic per workgroup; the host divides by 2^24 |Omega|.
namespace tgs {

__global__ void __launch_bounds__(256) view_error_sum_kernel(const uint16_t* __restrict__ E, int64_t pixels,
                                                             unsigned long long* __restrict__ sums) {
  __shared__ unsigned long long red[256];
  const int v = blockIdx.y;
  const uint16_t* map = E + (int64_t)v * pixels;
  unsigned long long acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pixels; i += (int64_t)gridDim.x * 256)
    acc += half_weight(map[i]);
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0 && red[0] != 0ull) atomicAdd(&sums[v], red[0]);
}

__global__ void __launch_bounds__(256) clear_u64_kernel(unsigned long long* __restrict__ p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

}  // namespace tgs

extern "C" int32_t tgs_view_error_sums(const uint16_t* E, int32_t n_views, int64_t pixels, uint64_t* sums,
                                       void* stream) {
  using namespace tgs;
  TGS_REQUIRE(n_views >= 0 && n_views <= 65535, "tgs_view_error_sums: n_views %d out of range", n_views);
  TGS_REQUIRE(pixels > 0 && pixels < (1ll << 31), "tgs_view_error_sums: pixels out of range");
  if (n_views == 0) return TGS_OK;
  TGS_REQUIRE(E && sums, "tgs_view_error_sums: null pointer");
  hipStream_t s = as_stream(stream);
  hipLaunchKernelGGL(clear_u64_kernel, dim3((unsigned)ceil_div(n_views, 256)), dim3(256), 0, s,
                     (unsigned long long*)sums, n_views);
  const unsigned bx = (unsigned)std::min<int64_t>(ceil_div(pixels, (int64_t)256 * 16), 256);
  hipLaunchKernelGGL(view_error_sum_kernel, dim3(bx, (unsigned)n_views), dim3(256), 0, s, E, pixels,
                     (unsigned long long*)sums);
  return hip_status("tgs_view_error_sums");
}
