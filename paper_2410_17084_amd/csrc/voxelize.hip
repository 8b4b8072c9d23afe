// vgpr_voxelize: the STORE step of Alg. S1 (paper supplementary) on the GPU.
//
// 1. key kernel: the packed 64-bit voxel key of every point (one IEEE double
//    multiply by 1/s and a floor per axis), the batch's index ranges, and the
//    call's counters cleared; non-finite points get the all-ones sentinel key.
// 2. compose kernel: the sort key, and the digit histograms of every pass. The
//    sort key is a compacted form of the voxel key with the same order: each
//    axis index minus the batch minimum, packed into just the bits the batch's
//    ranges need, then an invalid-point bit, then the frame index (a batch is
//    sorted by (frame, key)). A spinning scan needs ~24 key bits, so four
//    passes instead of eight. If the packed form does not fit 64 bits the
//    frame index gets its own extra passes, read from the point's index.
// 3. stable LSD radix sort of (sort key, index), 8-bit digits, one kernel a
//    pass: a tile's place among the tiles before it comes from their published
//    digit counts (decoupled look-back). Ranks inside a tile come from 64-lane
//    ballots, so equal digits keep their input order and the sort is stable.
// 4. segment kernel: voxel heads (key change or frame start), numbered by a
//    look-back of their counts; keys, starts, counts and frame ranges.
//
// The sort key's form stays on the device: four passes on 32-bit keys and the
// segmentation are launched at once, a pass that the form does not have leaves
// at once, and the host waits only for the results. For a form of more than 32
// bits these leave at once, and passes on 64-bit keys and their segmentation
// follow after that wait.
//
// Bound: up to ~300k points launches and waits, seven kernels' latencies of an uncached word
// each; above that the four passes (28 us each for 3.7M points, of which 12.6 us are their
// bytes, then tickets and the look-back). Whole calls, against a histogram, a scan and a
// scatter kernel a pass on 64-bit keys, four segmentation kernels, two copies and a wait for
// the key ranges: 16,384 points 104 -> 59 us, 131,072 117 -> 72, 524,288 134 -> 95, 64 frames
// of 57,600 273 -> 204.
#include <algorithm>
#include <climits>

#include "scan.h"
#include "vgpr_internal.h"

namespace vgpr {
namespace {

constexpr int kKeyThreads = 256;
constexpr int kKeyItems = 4;
constexpr int kKeyBlocks = 2048;                    // at most: every compose block reads all their partials
constexpr int kComposeThreads = 1024;
constexpr int kSmallCompose = 1, kLargeCompose = 2; // elements a thread reads together
constexpr int kComposeBlocks = 256;
constexpr int kSegItems = 8;
constexpr int kSmallSeg = 256, kLargeSeg = 1024;    // threads
constexpr int kMaxPasses = 12;                      // 8 of the packed key, 4 of the frame index
constexpr int kNarrowPasses = 4;                    // sort keys of 32 bits
// Tile of a sort pass: 1024 elements up to kSmallSort, where more tiles mean more CUs; 6144
// above, where fewer tiles mean fewer tickets and a shorter look-back. All passes of a call,
// 1024 against 6144: 131,072 points 29 / 38 us, 262,144 36 / 40, 524,288 55 / 43. At 3.7M
// points: 4096 115 us, 6144 111, 8192 127.
constexpr uint32_t kSmallSort = 1u << 18;
constexpr int kSmallThreads = 512, kSmallItems = 2;
constexpr int kLargeThreads = 1024, kLargeItems = 6;
constexpr int kWideThreads = 512, kWideItems = 8;

// Result words of a call, in pinned host memory: the kernels write them there.
enum { R_NVOX = 0, R_INVALID = 1, R_RANGE = 2, R_PASSES = 3, R_FRAMES = 4 };

// Compacted sort key: fields (k - kmin) in bx / by / bz bits (x highest), the
// invalid flag at bit B = bx + by + bz, the frame index above it if embedded.
// In Morton form the B field bits are interleaved instead (see interleave3), so
// that runs of consecutive voxels cover compact 3-D regions.
struct KeyForm {
  int bx, by, bz, B;
  int embed;           // frame index in bits [B + 1, ...)
  int key_passes;      // radix passes over the packed key
  int passes;          // and with those over the frame index; 0 if the call is refused
  int morton;          // field bits interleaved (1) or concatenated (0)
  int invalid, range;  // points that are not finite; whether one is out of the index range
  int64_t mn[3];       // per-axis minimum voxel index
};

// Morton interleave of fields of unequal widths: bit l of z, then of y, then
// of x, for l = 0, 1, ...; an axis drops out once l reaches its width, so the
// code takes exactly B bits and is a bijection of the three fields.
__device__ __forceinline__ uint64_t interleave3(uint64_t ux, uint64_t uy, uint64_t uz, const KeyForm& kf) {
  uint64_t tk = 0;
  int o = 0;
  const int top = max(kf.bx, max(kf.by, kf.bz));
  for (int l = 0; l < top; ++l) {
    if (l < kf.bz) tk |= ((uz >> l) & 1ull) << o++;
    if (l < kf.by) tk |= ((uy >> l) & 1ull) << o++;
    if (l < kf.bx) tk |= ((ux >> l) & 1ull) << o++;
  }
  return tk;
}

__device__ __forceinline__ void deinterleave3(uint64_t tk, const KeyForm& kf, uint64_t* ux, uint64_t* uy,
                                              uint64_t* uz) {
  uint64_t x = 0, y = 0, z = 0;
  int o = 0;
  const int top = max(kf.bx, max(kf.by, kf.bz));
  for (int l = 0; l < top; ++l) {
    if (l < kf.bz) z |= ((tk >> o++) & 1ull) << l;
    if (l < kf.by) y |= ((tk >> o++) & 1ull) << l;
    if (l < kf.bx) x |= ((tk >> o++) & 1ull) << l;
  }
  *ux = x;
  *uy = y;
  *uz = z;
}

__device__ __forceinline__ int frame_of(uint32_t idx, const int64_t* fo, int nf) {
  // largest f with fo[f] <= idx, for nf frames (fo has nf + 1 entries)
  int lo = 0, hi = nf - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (fo[mid] <= (int64_t)idx) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ uint32_t digit_of(uint64_t key, uint32_t val, int pass, int key_passes, const int64_t* fo,
                                             int nf) {
  if (pass < key_passes) return (uint32_t)(key >> (8 * pass)) & 0xFFu;
  return ((uint32_t)frame_of(val, fo, nf) >> (8 * (pass - key_passes))) & 0xFFu;
}

__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = min(v, __shfl_xor(v, d, 64));
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = max(v, __shfl_xor(v, d, 64));
  return v;
}

// Per-block results of the key kernel.
struct KeyPart {
  int mn[3], mx[3];
  int invalid, range;
};

// A grid-wide published word: tiles of one launch read each other's through these.
template <typename T>
__device__ __forceinline__ T peek(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void publish(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The next tile of a launch. Tiles are taken in the order in which their workgroups start, so
// the tiles before a running one have all started, and a wait for what they publish ends.
__device__ __forceinline__ uint32_t take_tile(uint32_t* ticket, uint32_t* smem) {
  if (threadIdx.x == 0) *smem = atomicAdd(ticket, 1u);
  __syncthreads();
  const uint32_t t = __builtin_amdgcn_readfirstlane(*smem);
  return t;
}

// Voxel key of every point (packed, biased), per-block index ranges and counts of unusable
// points. Also clears the `zero_words` words of the sort's counters and brings the frame
// offsets from pinned host memory: a memset and a copy would each be a launch of their own.
__global__ void __launch_bounds__(kKeyThreads) key_kernel(const float* __restrict__ xyz, uint32_t n, double inv_s,
                                                          uint64_t* __restrict__ keys, KeyPart* __restrict__ part,
                                                          uint32_t* __restrict__ zero, size_t zero_words,
                                                          const int64_t* __restrict__ h_fo, int64_t* __restrict__ fo,
                                                          int nf) {
  const size_t gid = (size_t)blockIdx.x * kKeyThreads + threadIdx.x;
  const size_t gsz = (size_t)gridDim.x * kKeyThreads;
  for (size_t j = gid; j < zero_words; j += gsz) zero[j] = 0u;
  if (nf == 1) {  // no read across the bus
    if (gid < 2) fo[gid] = gid ? (int64_t)n : 0;
  } else {
    for (size_t j = gid; j <= (size_t)nf; j += gsz) fo[j] = h_fo[j];
  }
  int invalid = 0, range = 0;
  int mn[3] = {INT_MAX, INT_MAX, INT_MAX}, mx[3] = {INT_MIN, INT_MIN, INT_MIN};
  for (size_t base = (size_t)blockIdx.x * kKeyThreads * kKeyItems; base < n; base += gsz * kKeyItems) {
    float c[kKeyItems][3];
#pragma unroll
    for (int r = 0; r < kKeyItems; ++r) {
      const size_t i = base + r * kKeyThreads + threadIdx.x;
#pragma unroll
      for (int a = 0; a < 3; ++a) c[r][a] = i < n ? xyz[3 * i + a] : 0.0f;
    }
#pragma unroll
    for (int r = 0; r < kKeyItems; ++r) {
      const size_t i = base + r * kKeyThreads + threadIdx.x;
      if (i >= n) continue;
      uint64_t key = kKeySentinel;
      if (isfinite(c[r][0]) && isfinite(c[r][1]) && isfinite(c[r][2])) {
        double k[3];
        bool in = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          k[a] = floor(__dmul_rn((double)c[r][a], inv_s));
          in = in && !(fabs(k[a]) > (double)kKeyAxisLimit);
        }
        if (in) {
          key = 0;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const int ia = (int)k[a];
            mn[a] = min(mn[a], ia);
            mx[a] = max(mx[a], ia);
            key = (key << kKeyFieldBits) | (uint64_t)((int64_t)ia + kKeyBias);
          }
        } else {
          range = 1;
        }
      } else {
        ++invalid;
      }
      keys[i] = key;
    }
  }
  __shared__ int s[8][kKeyThreads / 64];
  const int w = threadIdx.x >> 6;
  int red[8] = {wave_min_i(mn[0]), wave_min_i(mn[1]), wave_min_i(mn[2]), wave_max_i(mx[0]), wave_max_i(mx[1]),
                wave_max_i(mx[2]), (int)wave_sum((uint32_t)invalid), wave_max_i(range)};
  if (lane_id() == 0) {
#pragma unroll
    for (int a = 0; a < 8; ++a) s[a][w] = red[a];
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    const int a = threadIdx.x;
    int r = s[a][0];
    for (int k = 1; k < kKeyThreads / 64; ++k) {
      const int v = s[a][k];
      r = a < 3 ? min(r, v) : a == 6 ? r + v : max(r, v);
    }
    reinterpret_cast<int*>(part + blockIdx.x)[a] = r;
  }
}

__device__ __forceinline__ int bits_of(int64_t r) { return r > 0 ? 64 - __clzll(r) : 0; }

// The batch's sort key form, from the key kernel's partials; every thread of the block gets it.
template <int NT>
__device__ KeyForm key_form(const KeyPart* __restrict__ part, int nparts, uint32_t n, int nf, int morton) {
  __shared__ int s[8][NT / 64];
  int v[8] = {INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN, 0, 0};
  for (int b = threadIdx.x; b < nparts; b += NT) {
    const KeyPart p = part[b];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = min(v[a], p.mn[a]);
      v[3 + a] = max(v[3 + a], p.mx[a]);
    }
    v[6] += p.invalid;
    v[7] |= p.range;
  }
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int r = a < 3 ? wave_min_i(v[a]) : a == 6 ? (int)wave_sum((uint32_t)v[a]) : wave_max_i(v[a]);
    if (lane_id() == 0) s[a][threadIdx.x >> 6] = r;
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    int r = s[a][0];
#pragma unroll
    for (int k = 1; k < NT / 64; ++k) r = a < 3 ? min(r, s[a][k]) : a == 6 ? r + s[a][k] : max(r, s[a][k]);
    v[a] = __builtin_amdgcn_readfirstlane(r);
  }
  KeyForm kf{};
  kf.invalid = v[6];
  kf.range = v[7];
  const bool any_valid = (uint32_t)v[6] < n;
  int b3[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    kf.mn[a] = any_valid ? v[a] : 0;
    b3[a] = any_valid ? bits_of((int64_t)v[3 + a] - v[a]) : 0;
  }
  kf.bx = b3[0];
  kf.by = b3[1];
  kf.bz = b3[2];
  kf.B = b3[0] + b3[1] + b3[2];
  const int bf = nf > 1 ? bits_of(nf - 1) : 0;
  kf.embed = kf.B + 1 + bf <= 64 ? 1 : 0;
  kf.key_passes = (kf.B + 1 + (kf.embed ? bf : 0) + 7) / 8;
  kf.passes = v[7] ? 0 : kf.key_passes + (kf.embed ? 0 : (bf + 7) / 8);
  kf.morton = morton;
  return kf;
}

__device__ __forceinline__ uint64_t pack_sort_key(uint64_t key, const KeyForm& kf) {
  if (key == kKeySentinel) return 1ull << kf.B;
  const int64_t mask = (int64_t(1) << kKeyFieldBits) - 1;
  const uint64_t ux = (uint64_t)((int64_t)((key >> (2 * kKeyFieldBits)) & mask) - kKeyBias - kf.mn[0]);
  const uint64_t uy = (uint64_t)((int64_t)((key >> kKeyFieldBits) & mask) - kKeyBias - kf.mn[1]);
  const uint64_t uz = (uint64_t)((int64_t)(key & mask) - kKeyBias - kf.mn[2]);
  return kf.morton ? interleave3(ux, uy, uz, kf) : (ux << (kf.by + kf.bz)) | (uy << kf.bz) | uz;
}

// Packed key -> compacted sort key, and every pass's digit histogram. Keys of up to 32 bits go
// to `narrow`, wider ones stay in place. A scan's neighbours often share their digits, and
// LDS adds to one word go one by one: only the first lane of a run adds, with its length.
template <int ITEMS>
__global__ void __launch_bounds__(kComposeThreads) compose_kernel(
    uint64_t* __restrict__ keys, uint32_t* __restrict__ narrow, uint32_t n, const KeyPart* __restrict__ part, int nparts,
    int morton, const int64_t* __restrict__ fo, int nf, KeyForm* __restrict__ form, uint32_t* __restrict__ hist) {
  constexpr int kTile = kComposeThreads * ITEMS;
  __shared__ uint32_t h[kMaxPasses * 256];
  const KeyForm kf = key_form<kComposeThreads>(part, nparts, n, nf, morton);
  if (blockIdx.x == 0 && threadIdx.x == 0) *form = kf;
  if (kf.range) return;
  for (int j = threadIdx.x; j < kf.passes * 256; j += kComposeThreads) h[j] = 0;
  __syncthreads();
  // a block's elements are consecutive, so its frames are too
  const size_t tiles = ((size_t)n + kTile - 1) / kTile;
  const size_t b0 = tiles * blockIdx.x / gridDim.x * kTile;
  const size_t b1 = tiles * (blockIdx.x + 1) / gridDim.x * kTile;
  const bool frames = kf.embed && nf > 1;
  int f = frames ? frame_of((uint32_t)(b0 < n ? b0 : n - 1), fo, nf) : 0;
  const unsigned long long upto = ~0ull >> (63 - lane_id());
  for (size_t base = b0; base < b1; base += kTile) {
    uint64_t k[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const size_t i = base + r * kComposeThreads + threadIdx.x;
      k[r] = i < n ? keys[i] : kKeySentinel;
    }
    if (frames && fo[f + 1] <= (int64_t)base) f = frame_of((uint32_t)(base < n ? base : n - 1), fo, nf);
    const int64_t frame_end = frames ? fo[f + 1] : 0;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const size_t i = base + r * kComposeThreads + threadIdx.x;
      const bool in = i < n;
      uint64_t tk = pack_sort_key(k[r], kf);
      if (frames && in)
        tk |= (uint64_t)((int64_t)i < frame_end ? f : frame_of((uint32_t)i, fo, nf)) << (kf.B + 1);
      if (in) {
        if (kf.passes <= kNarrowPasses) narrow[i] = (uint32_t)tk;
        else keys[i] = tk;
      }
      const unsigned long long act = __ballot(in);
      for (int p = 0; p < kf.passes; ++p) {
        const uint32_t d = in ? digit_of(tk, (uint32_t)i, p, kf.key_passes, fo, nf) : 256u;
        const uint32_t prev = __shfl_up(d, 1, 64);
        const bool first = lane_id() == 0 || prev != d;
        const unsigned long long heads = __ballot(first);
        if (first && in) {
          const unsigned long long after = heads & ~upto;
          const int end = after ? __ffsll(after) - 1 : __popcll(act);
          atomicAdd(&h[p * 256 + d], (uint32_t)(end - lane_id()));
        }
      }
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < kf.passes * 256; j += kComposeThreads) {
    const uint32_t c = h[j];
    if (c) atomicAdd(&hist[j], c);
  }
}

// Compacted sort key -> packed voxel key.
__device__ __forceinline__ uint64_t unpack_sort_key(uint64_t tk, const KeyForm& kf) {
  if (kf.morton) {
    uint64_t ux, uy, uz;
    deinterleave3(tk, kf, &ux, &uy, &uz);
    return ((uint64_t)((int64_t)ux + kf.mn[0] + kKeyBias) << (2 * kKeyFieldBits)) |
           ((uint64_t)((int64_t)uy + kf.mn[1] + kKeyBias) << kKeyFieldBits) | (uint64_t)((int64_t)uz + kf.mn[2] + kKeyBias);
  }
  const uint64_t mz = (kf.bz ? (1ull << kf.bz) : 1ull) - 1ull, my = (kf.by ? (1ull << kf.by) : 1ull) - 1ull,
                 mx = (kf.bx ? (1ull << kf.bx) : 1ull) - 1ull;
  const int64_t kz = (int64_t)(tk & mz) + kf.mn[2];
  const int64_t ky = (int64_t)((tk >> kf.bz) & my) + kf.mn[1];
  const int64_t kx = (int64_t)((tk >> (kf.by + kf.bz)) & mx) + kf.mn[0];
  return ((uint64_t)(kx + kKeyBias) << (2 * kKeyFieldBits)) | ((uint64_t)(ky + kKeyBias) << kKeyFieldBits) |
         (uint64_t)(kz + kKeyBias);
}

// What tiles publish for one digit. A tile: 0 until known, then its count + 1. A group of 16
// tiles: the sum of their counts, with the number of tiles in it from bit 24. A group with all
// before it: 0 until known, then the count with the top bit. A tile adds up the tiles before
// it in its group and the groups before that, 16 words of a digit at a time: with single tiles
// alone the last of 450 tiles walks 28 steps of an uncached read (~0.5 us), with groups three.
constexpr uint32_t kInclusive = 0x80000000u;
constexpr int kGroup = 16;

struct Published {
  uint32_t *tiles, *groups, *upto;  // rows of 256 digits
};

__host__ __device__ __forceinline__ size_t published_rows(uint32_t max_tiles) {
  return (size_t)max_tiles + 2 * ((size_t)(max_tiles + kGroup - 1) / kGroup);
}

__device__ __forceinline__ Published published(uint32_t* status, int half, uint32_t max_tiles) {
  uint32_t* t = status + half * published_rows(max_tiles) * 256;
  uint32_t* g = t + (size_t)max_tiles * 256;
  return {t, g, g + (size_t)((max_tiles + kGroup - 1) / kGroup) * 256};
}

// Digit `d`'s elements in the tiles before `tile`.
__device__ __forceinline__ uint32_t before_tile(const Published& pub, uint32_t tile, int d) {
  const uint32_t group = tile / kGroup, in_group = tile % kGroup;
  uint32_t excl = 0;
  {
    const uint32_t* rows = pub.tiles + (size_t)group * kGroup * 256 + d;
    uint32_t w[kGroup - 1];
#pragma unroll
    for (int j = 0; j < kGroup - 1; ++j) w[j] = j < (int)in_group ? peek(rows + 256 * j) : 1u;
#pragma unroll
    for (int j = 0; j < kGroup - 1; ++j) {
      while (w[j] == 0u) {
        __builtin_amdgcn_s_sleep(1);
        w[j] = peek(rows + 256 * j);
      }
      excl += w[j] - 1u;
    }
  }
  for (int64_t g = (int64_t)group - 1; g >= 0; g -= kGroup) {
    // groups g, g - 1, .. ; the farthest is asked for the prefix it closes
    const int64_t far = g - (kGroup - 1) > 0 ? g - (kGroup - 1) : 0;
    uint32_t w[kGroup];
    const uint32_t up = peek(pub.upto + (size_t)far * 256 + d);
#pragma unroll
    for (int j = 0; j < kGroup; ++j) w[j] = g - j >= 0 ? peek(pub.groups + (size_t)(g - j) * 256 + d) : 0u;
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
      if (g - j < 0 || (g - j == far && up)) continue;
      while ((w[j] >> 24) != kGroup) {
        __builtin_amdgcn_s_sleep(1);
        w[j] = peek(pub.groups + (size_t)(g - j) * 256 + d);
      }
      excl += w[j] & 0xFFFFFFu;
    }
    if (up) {
      excl += up & ~kInclusive;
      break;
    }
  }
  return excl;
}

// One radix pass. Element order inside a tile is (wave, round, lane), which is the input
// order, so ranks from ballots preserve stability. The tile is put in order in LDS first, so
// the stores of a digit's run are consecutive. Pass p's words are in half p & 1; it clears
// the other half, which pass p - 1 is done with, for pass p + 1.
template <typename K, int NT, int ITEMS>
__global__ void __launch_bounds__(NT) radix_pass(K* __restrict__ keys_a, K* __restrict__ keys_b,
                                                 uint32_t* __restrict__ perm, uint32_t* __restrict__ vals_tmp,
                                                 uint32_t n, int pass, const KeyForm* __restrict__ form,
                                                 const int64_t* __restrict__ fo, int nf,
                                                 const uint32_t* __restrict__ hist, uint32_t* __restrict__ status,
                                                 uint32_t max_tiles, uint32_t* __restrict__ tickets) {
  constexpr bool kNarrow = sizeof(K) == 4;
  constexpr int kWaves = NT / 64;
  constexpr uint32_t kTile = NT * ITEMS;
  __shared__ uint32_t cnt[kWaves][256];
  __shared__ uint32_t scan_smem[kWaves + 1];
  __shared__ uint32_t gbase[256];
  __shared__ K skey[kTile];
  __shared__ uint32_t sval[kTile];
  __shared__ uint32_t s_tile;
  const int passes = form->passes, key_passes = form->key_passes;
  if (pass >= passes || (passes <= kNarrowPasses) != kNarrow) return;
  const K* __restrict__ keys_in = (pass & 1) ? keys_b : keys_a;
  K* __restrict__ keys_out = (pass & 1) ? keys_a : keys_b;
  // the last pass writes the indices into perm; pass 0 reads none (element i is point i)
  const bool to_perm = ((passes - 1 - pass) & 1) == 0;
  const uint32_t* vals_in = to_perm ? vals_tmp : perm;
  uint32_t* vals_out = to_perm ? perm : vals_tmp;
  auto digit = [&](K key, uint32_t val) -> uint32_t {
    if (kNarrow) return (uint32_t)(key >> (8 * pass)) & 0xFFu;
    return digit_of(key, val, pass, key_passes, fo, nf);
  };
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;

  for (int i = tid; i < kWaves * 256; i += NT) (&cnt[0][0])[i] = 0;
  const uint32_t tile = take_tile(&tickets[pass], &s_tile);
  const Published pub = published(status, pass & 1, max_tiles);
  const uint32_t group = tile / kGroup;
  if (tid < 256) {
    const Published next = published(status, (pass + 1) & 1, max_tiles);
    next.tiles[(size_t)tile * 256 + tid] = 0;
    if (tile % kGroup == 0) next.groups[(size_t)group * 256 + tid] = next.upto[(size_t)group * 256 + tid] = 0;
  }

  const uint32_t base = tile * kTile + wave * 64 * ITEMS;
  K k[ITEMS];
  uint32_t v[ITEMS], old[ITEMS], rank[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t i = base + r * 64 + lane;
    k[r] = i < n ? keys_in[i] : K(0);
    v[r] = i < n ? (pass ? vals_in[i] : i) : 0u;
  }
  // global start of each digit
  uint32_t dtot;
  const uint32_t digit_start = block_exclusive_sum<NT>(tid < 256 ? hist[pass * 256 + tid] : 0u, scan_smem,
                                                                 &dtot);
  // A wave's rounds one after another: the first lane of each digit adds the round's count to
  // the wave's counter. The adds need no answer until all are issued.
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  uint32_t from[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool valid = base + r * 64 + lane < n;
    const uint32_t d = valid ? digit(k[r], v[r]) : 0u;
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const unsigned long long bal = __ballot(valid && bit);
      peers &= bit ? bal : ~bal;
    }
    rank[r] = (uint32_t)__popcll(peers & lt_mask);
    from[r] = valid ? (uint32_t)__ffsll(peers) - 1u : 0u;
    old[r] = 0;
    if (valid && rank[r] == 0) old[r] = atomicAdd(&cnt[wave][d], (uint32_t)__popcll(peers));
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) rank[r] += __shfl(old[r], from[r], 64);
  __syncthreads();
  uint32_t sum = 0;
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t c = cnt[w][tid];
      cnt[w][tid] = sum;
      sum += c;
    }
    publish(&pub.tiles[(size_t)tile * 256 + tid], sum + 1u);
    atomicAdd(&pub.groups[(size_t)group * 256 + tid], sum + (1u << 24));
  }
  const uint32_t local = block_exclusive_sum<NT>(sum, scan_smem, &dtot);
  if (tid < 256) {
    const uint32_t excl = before_tile(pub, tile, tid);
    if (tile % kGroup == kGroup - 1) publish(&pub.upto[(size_t)group * 256 + tid], kInclusive | (excl + sum));
    gbase[tid] = digit_start + excl - local;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) cnt[w][tid] += local;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    if (base + r * 64 + lane < n) {
      const uint32_t p = cnt[wave][digit(k[r], v[r])] + rank[r];
      skey[p] = k[r];
      sval[p] = v[r];
    }
  }
  __syncthreads();
  const uint32_t have = min(kTile, n - tile * kTile);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t p = r * NT + tid;
    if (p < have) {
      const K kk = skey[p];
      const uint32_t vv = sval[p];
      const uint32_t dst = gbase[digit(kk, vv)] + p;
      if (dst < n) {
        keys_out[dst] = kk;
        vals_out[dst] = vv;
      }
    }
  }
}

__device__ __forceinline__ bool sort_key_valid(uint64_t k, const KeyForm& kf) { return ((k >> kf.B) & 1ull) == 0; }

// Whether sorted elements i - 1 and i, with keys a and b, are of one voxel (b is a valid one).
__device__ __forceinline__ bool same_voxel(uint64_t a, uint64_t b, uint32_t i, const KeyForm& kf, const int64_t* fo,
                                           int nf) {
  if (a != b) return false;
  return kf.embed || nf == 1 || frame_of(i, fo, nf) == frame_of(i - 1, fo, nf);
}

// A tile's published word of the segmentation: 0 until known, then bit 62 (the tile alone) or
// bit 63 (with all before it), the voxel heads in bits 31..61 and the last head's position + 1
// in bits 0..30 (0: no head).
constexpr unsigned long long kSegAlone = 1ull << 62, kSegUpTo = 1ull << 63, kSegPos = (1ull << 31) - 1;

// Voxel heads are numbered in order; the voxel's last element writes its count, with the
// head's position from the tile's own list or from the look-back. Frame f's first voxel is
// the number of heads before element fo[f].
template <typename K, int NT>
__global__ void __launch_bounds__(NT) segment_kernel(
    const K* __restrict__ keys_a, const K* __restrict__ keys_b, uint32_t n, const KeyForm* __restrict__ form,
    const int64_t* __restrict__ fo, int nf, unsigned long long* __restrict__ status,
    uint32_t ntiles, uint32_t* __restrict__ ticket, int64_t cap, uint64_t* __restrict__ out_keys,
    int32_t* __restrict__ out_off, int32_t* __restrict__ out_cnt, unsigned long long* __restrict__ h_res) {
  constexpr int kTile = NT * kSegItems;
  __shared__ uint32_t scan_smem[NT / 64 + 1];
  __shared__ uint32_t pos[kTile];
  __shared__ uint32_t s_tile;
  __shared__ unsigned long long s_before;
  const KeyForm kf = *form;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    h_res[R_INVALID] = (unsigned long long)kf.invalid;
    h_res[R_RANGE] = (unsigned long long)kf.range;
    h_res[R_PASSES] = (unsigned long long)kf.passes;
  }
  if (kf.passes == 0 || (kf.passes <= kNarrowPasses) != (sizeof(K) == 4)) return;
  const K* __restrict__ keys = (kf.passes & 1) ? keys_b : keys_a;
  const int tid = threadIdx.x;
  const uint32_t tile = take_tile(ticket, &s_tile);
  const uint32_t t0 = tile * kTile;
  const uint32_t first = t0 + tid * kSegItems;
  // a thread's elements are consecutive, with one on either side
  uint64_t k[kSegItems + 2];
#pragma unroll
  for (int r = 0; r < kSegItems + 2; ++r) {
    const uint32_t i = first + r - 1;  // wraps below element 0
    k[r] = i < n ? keys[i] : 0ull;
  }
  uint32_t head = 0, tail = 0;  // bit r: element first + r
#pragma unroll
  for (int r = 0; r < kSegItems; ++r) {
    const uint32_t i = first + r;
    if (i < n && sort_key_valid(k[r + 1], kf)) {
      if (i == 0 || !same_voxel(k[r], k[r + 1], i, kf, fo, nf)) head |= 1u << r;
      if (i == n - 1 || !same_voxel(k[r + 1], k[r + 2], i + 1, kf, fo, nf)) tail |= 1u << r;
    }
  }
  uint32_t heads;
  const uint32_t ex = block_exclusive_sum<NT>((uint32_t)__popc(head), scan_smem, &heads);
  {
    uint32_t o = ex;
#pragma unroll
    for (int r = 0; r < kSegItems; ++r)
      if (head >> r & 1u) pos[o++] = first + r;
  }
  __syncthreads();
  if (tid < 64) {
    const unsigned long long own = ((unsigned long long)heads << 31) | (heads ? pos[heads - 1] + 1ull : 0ull);
    if (tid == 0) publish(&status[tile], (tile == 0 ? kSegUpTo : kSegAlone) | own);
    // the 64 tiles before, then the 64 before those, until one that holds its own prefix
    unsigned long long count = 0, last = 0;
    int64_t back = (int64_t)tile - 1;
    while (back >= 0) {
      const int64_t t = back - tid;
      unsigned long long w;
      unsigned long long up;
      do {
        w = t >= 0 ? peek(&status[t]) : kSegUpTo;
        up = __ballot((w & kSegUpTo) != 0);
        // lanes past the first prefix are not needed
        const unsigned long long need = up ? ((up & -up) << 1) - 1ull : ~0ull;
        if ((__ballot(w != 0) & need) == need) break;
        __builtin_amdgcn_s_sleep(1);
      } while (true);
      const int stop = up ? __ffsll(up) - 1 : 63;
      unsigned long long c = tid <= stop ? (w >> 31) & kSegPos : 0ull;
      unsigned long long p = tid <= stop ? w & kSegPos : 0ull;  // positions grow with the tile: the maximum is the last
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        c += __shfl_xor(c, d, 64);
        const unsigned long long q = __shfl_xor(p, d, 64);
        p = q > p ? q : p;
      }
      count += c;
      last = p > last ? p : last;
      if (up) break;
      back -= 64;
    }
    if (tid == 0) {
      const unsigned long long all = ((count + heads) << 31) | (heads ? own & kSegPos : last);
      if (tile) publish(&status[tile], kSegUpTo | all);
      s_before = (count << 31) | last;
      if (tile == ntiles - 1) h_res[R_NVOX] = count + heads;
    }
  }
  __syncthreads();
  const uint32_t vbase = (uint32_t)(s_before >> 31);
  uint32_t o = ex;  // heads of the tile before element first + r
#pragma unroll
  for (int r = 0; r < kSegItems; ++r) {
    const uint32_t i = first + r;
    if (head >> r & 1u) {
      const uint32_t vid = vbase + o++;
      if ((int64_t)vid < cap) {
        out_keys[vid] = unpack_sort_key(k[r + 1], kf);
        out_off[vid] = (int32_t)i;
      }
    }
    if (tail >> r & 1u) {
      const uint32_t vid = vbase + o - 1;
      const uint32_t start = o ? pos[o - 1] : (uint32_t)(s_before & kSegPos) - 1u;
      if ((int64_t)vid < cap) out_cnt[vid] = (int32_t)(i + 1 - start);
    }
  }
  // frames that start in this tile; the last tile also has those that start at n
  const int64_t end = tile == ntiles - 1 ? (int64_t)n + 1 : (int64_t)t0 + kTile;
  int lo = 0, hi = nf + 1;  // first f with fo[f] >= t0
  while (lo < hi) {
    const int m = (lo + hi) >> 1;
    if (fo[m] < (int64_t)t0) lo = m + 1; else hi = m;
  }
  for (int64_t f = (int64_t)lo + tid; f <= nf && fo[f] < end; f += NT) {
    const int64_t target = fo[f];
    uint32_t a = 0, b = heads;  // heads of the tile before the target
    while (a < b) {
      const uint32_t m = (a + b) >> 1;
      if ((int64_t)pos[m] < target) a = m + 1; else b = m;
    }
    h_res[R_FRAMES + f] = (unsigned long long)vbase + a;
  }
}

}  // namespace

vgpr_status voxelize_impl(vgpr_ctx* ctx, const float* d_xyz, int64_t n_pts, const int64_t* h_frame_offsets,
                          int32_t n_frames, float voxel_size, uint64_t* d_keys, int32_t* d_offsets,
                          int32_t* d_counts, int32_t* d_perm, int64_t cap_vox, int64_t* h_n_vox,
                          int64_t* h_frame_vox, int64_t* h_n_invalid, size_t work_offset, bool morton) {
  if (n_pts < 0 || n_pts >= (int64_t(1) << 31)) return fail(ctx, VGPR_E_INVALID, "n_pts out of range");
  if (cap_vox < 0) return fail(ctx, VGPR_E_INVALID, "cap_vox < 0");
  if (!h_n_vox) return fail(ctx, VGPR_E_INVALID, "h_n_vox is NULL");
  if (n_pts > 0 && (!d_xyz || !d_perm)) return fail(ctx, VGPR_E_INVALID, "d_xyz / d_perm is NULL");
  if (cap_vox > 0 && (!d_keys || !d_offsets || !d_counts))
    return fail(ctx, VGPR_E_INVALID, "voxel output buffer is NULL");
  const int nf = n_frames < 1 ? 1 : n_frames;
  std::vector<int64_t> fo(nf + 1, 0);
  if (h_frame_offsets && n_frames >= 1) {
    for (int f = 0; f <= nf; ++f) fo[f] = h_frame_offsets[f];
    if (fo[0] != 0 || fo[nf] != n_pts) return fail(ctx, VGPR_E_INVALID, "frame offsets must span [0, n_pts]");
    for (int f = 0; f < nf; ++f)
      if (fo[f + 1] < fo[f]) return fail(ctx, VGPR_E_INVALID, "frame offsets must be ascending");
  } else {
    if (n_frames > 1) return fail(ctx, VGPR_E_INVALID, "h_frame_offsets is NULL with n_frames > 1");
    fo[1] = n_pts;
  }
  const uint32_t n = (uint32_t)n_pts;
  const size_t res_words = R_FRAMES + (size_t)nf + 1;
  struct Layout {
    uint32_t max_tiles, nseg, kblocks;
    size_t o_hist, o_ticket, o_status, zero_words, words, need;
  };
  auto layout = [&](bool small) {
    Layout l{};
    const uint32_t min_tile =
        small ? kSmallThreads * kSmallItems : std::min(kLargeThreads * kLargeItems, kWideThreads * kWideItems);
    l.max_tiles = (uint32_t)((n_pts + min_tile - 1) / min_tile);
    const int seg_tile = kSegItems * (small ? kSmallSeg : kLargeSeg);
    l.nseg = (uint32_t)((n_pts + seg_tile - 1) / seg_tile);
    l.kblocks = (uint32_t)std::min<int64_t>((n_pts + kKeyThreads * kKeyItems - 1) / (kKeyThreads * kKeyItems), kKeyBlocks);
    // words cleared by the key kernel: segmentation look-back, histograms, tickets, the first pass's look-back
    l.o_hist = 2 * (size_t)l.nseg;
    l.o_ticket = l.o_hist + 256 * kMaxPasses;
    l.o_status = l.o_ticket + kMaxPasses + 2;
    l.zero_words = l.o_status + 256 * published_rows(l.max_tiles);
    l.words = l.zero_words + 256 * published_rows(l.max_tiles);
    l.need = work_offset + Carver::round(sizeof(uint64_t) * (size_t)n) * 2 + Carver::round(sizeof(uint32_t) * (size_t)n) +
             Carver::round(sizeof(uint32_t) * l.words) + Carver::round(sizeof(KeyPart) * (size_t)l.kblocks) +
             Carver::round(sizeof(int64_t) * ((size_t)nf + 1)) + Carver::round(sizeof(KeyForm)) + 4096;
    return l;
  };
  bool small = n <= kSmallSort;
  Layout lay = layout(small);
  // small tiles publish more (22.4 bytes a point, large ones 20.6): not where that is over an HBM budget
  if (small && ctx->budget && lay.need > ctx->work.bytes && ctx->held - ctx->work.bytes + lay.need > ctx->budget)
    lay = layout(small = false);
  const uint32_t max_tiles = lay.max_tiles, nseg = lay.nseg, kblocks = lay.kblocks;
  const size_t o_hist = lay.o_hist, o_ticket = lay.o_ticket, o_status = lay.o_status, zero_words = lay.zero_words,
               words = lay.words, need = lay.need;
  vgpr_status st = reserve_work(ctx, need);
  if (st != VGPR_OK) return st;
  st = reserve_pinned(ctx, sizeof(int64_t) * ((size_t)nf + 1) + sizeof(unsigned long long) * res_words + 64);
  if (st != VGPR_OK) return st;
  Carver cv(static_cast<char*>(ctx->work.ptr) + work_offset);
  uint64_t* keys_a = cv.take<uint64_t>(n);
  uint64_t* keys_b = cv.take<uint64_t>(n);
  uint32_t* vals_tmp = cv.take<uint32_t>(n);
  uint32_t* zero = cv.take<uint32_t>(words);
  KeyPart* part = cv.take<KeyPart>(kblocks);
  int64_t* d_fo = cv.take<int64_t>((size_t)nf + 1);
  KeyForm* form = cv.take<KeyForm>(1);

  int64_t* h_fo = static_cast<int64_t*>(ctx->pinned);
  unsigned long long* h_res = reinterpret_cast<unsigned long long*>(h_fo + nf + 1);
  std::copy(fo.begin(), fo.end(), h_fo);
  std::fill(h_res, h_res + res_words, 0ull);

  uint32_t* perm = reinterpret_cast<uint32_t*>(d_perm);
  uint32_t* narrow = reinterpret_cast<uint32_t*>(keys_b);  // its two halves, while keys_a has the packed keys
  auto pass = [&](auto kernel, int threads, uint32_t per_tile, auto* a, auto* b, int p) {
    hipLaunchKernelGGL(kernel, dim3((n + per_tile - 1) / per_tile), dim3(threads), 0, ctx->stream, a, b, perm, vals_tmp,
                       n, p, form, d_fo, nf, zero + o_hist, zero + o_status, max_tiles, zero + o_ticket);
  };
  auto segment = [&](auto kernel, auto* a, auto* b) {
    ProfScope ps(ctx, "voxelize_segment");
    hipLaunchKernelGGL(kernel, dim3(nseg), dim3(small ? kSmallSeg : kLargeSeg), 0, ctx->stream, a, b, n, form, d_fo, nf,
                       reinterpret_cast<unsigned long long*>(zero), nseg, zero + o_ticket + kMaxPasses, cap_vox, d_keys,
                       d_offsets, d_counts, h_res);
  };
  if (n > 0) {
    {
      ProfScope ps(ctx, "voxelize_key");
      hipLaunchKernelGGL(key_kernel, dim3(kblocks), dim3(kKeyThreads), 0, ctx->stream, d_xyz, n,
                         1.0 / (double)voxel_size, keys_a, part, zero, zero_words, h_fo, d_fo, nf);
      auto compose = [&](auto kernel, uint32_t per_block) {
        hipLaunchKernelGGL(kernel, dim3(std::min<uint32_t>((n + per_block - 1) / per_block, kComposeBlocks)),
                           dim3(kComposeThreads), 0, ctx->stream, keys_a, narrow, n, part, (int)kblocks, morton ? 1 : 0,
                           d_fo, nf, form, zero + o_hist);
      };
      if (small) compose(compose_kernel<kSmallCompose>, kComposeThreads * kSmallCompose);
      else compose(compose_kernel<kLargeCompose>, kComposeThreads * kLargeCompose);
    }
    {
      ProfScope ps(ctx, "voxelize_sort");
      for (int p = 0; p < kNarrowPasses; ++p) {
        if (small)
          pass(radix_pass<uint32_t, kSmallThreads, kSmallItems>, kSmallThreads, kSmallThreads * kSmallItems, narrow,
               narrow + n, p);
        else
          pass(radix_pass<uint32_t, kLargeThreads, kLargeItems>, kLargeThreads, kLargeThreads * kLargeItems, narrow,
               narrow + n, p);
      }
    }
    if (small) segment(segment_kernel<uint32_t, kSmallSeg>, narrow, narrow + n);
    else segment(segment_kernel<uint32_t, kLargeSeg>, narrow, narrow + n);
    VGPR_HIP(ctx, hipGetLastError());
  }
  VGPR_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (h_res[R_RANGE]) return fail(ctx, VGPR_E_RANGE, "a point's voxel index is outside +-(2^20 - 1)");
  const int passes = (int)h_res[R_PASSES];
  if (passes > kNarrowPasses) {
    {
      ProfScope ps(ctx, "voxelize_sort");
      for (int p = 0; p < passes; ++p) {
        if (small)
          pass(radix_pass<uint64_t, kSmallThreads, kSmallItems>, kSmallThreads, kSmallThreads * kSmallItems, keys_a,
               keys_b, p);
        else
          pass(radix_pass<uint64_t, kWideThreads, kWideItems>, kWideThreads, kWideThreads * kWideItems, keys_a, keys_b,
               p);
      }
    }
    if (small) segment(segment_kernel<uint64_t, kSmallSeg>, keys_a, keys_b);
    else segment(segment_kernel<uint64_t, kLargeSeg>, keys_a, keys_b);
    VGPR_HIP(ctx, hipGetLastError());
    VGPR_HIP(ctx, hipStreamSynchronize(ctx->stream));
  }
  const int64_t nvox = (int64_t)h_res[R_NVOX];
  *h_n_vox = nvox;
  if (h_n_invalid) *h_n_invalid = (int64_t)h_res[R_INVALID];
  if (nvox > cap_vox)
    return fail(ctx, VGPR_E_CAPACITY, "voxel count " + std::to_string(nvox) + " exceeds cap_vox");
  if (h_frame_vox)
    for (int f = 0; f <= nf; ++f) h_frame_vox[f] = n > 0 ? (int64_t)h_res[R_FRAMES + f] : 0;
  return VGPR_OK;
}

}  // namespace vgpr

extern "C" vgpr_status vgpr_voxelize(vgpr_ctx* ctx, const float* d_xyz, int64_t n_pts, const int64_t* h_frame_offsets,
                                     int32_t n_frames, const vgpr_params* params, uint64_t* d_keys,
                                     int32_t* d_offsets, int32_t* d_counts, int32_t* d_perm, int64_t cap_vox,
                                     int64_t* h_n_vox, int64_t* h_frame_vox, int64_t* h_n_invalid) {
  if (!ctx) return VGPR_E_INVALID;
  vgpr_status st = vgpr::check_params(ctx, params);
  if (st != VGPR_OK) return st;
  if (hipSetDevice(ctx->device) != hipSuccess) return vgpr::fail(ctx, VGPR_E_DEVICE, "hipSetDevice");
  return vgpr::voxelize_impl(ctx, d_xyz, n_pts, h_frame_offsets, n_frames, params->voxel_size, d_keys, d_offsets,
                             d_counts, d_perm, cap_vox, h_n_vox, h_frame_vox, h_n_invalid, 0);
}
