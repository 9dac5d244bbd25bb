// Device primitives: exclusive scan of int32 counts (three-pass, int64
// carries), integer max reduction and fills.
#include <algorithm>
#include <chrono>
#include <cstring>

#include "common.h"

namespace ppe {
namespace {

constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

__device__ __forceinline__ long long wave_incl_scan(long long v) {
  const int lane = threadIdx.x % kWave;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    long long u = __shfl_up(v, o, kWave);
    if (lane >= o) v += u;
  }
  return v;
}

// Exclusive scan across a block of kBlock threads; *total receives the sum.
__device__ __forceinline__ long long block_excl_scan(long long v, long long* total) {
  __shared__ long long wsum[kBlock / kWave];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  long long inc = wave_incl_scan(v);
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  long long off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kBlock / kWave; ++i) {
    if (i < w) off += wsum[i];
    tot += wsum[i];
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

// Read-back staging: item k (kPubMax at most) is off[k+1] - off[k] words at
// src[k], copied to dst[1 + off[k]..] in the pinned host box (dst null: nothing
// to publish).
constexpr int kPubMax = 16;
struct PubArgs {
  const uint32_t* src[kPubMax];
  uint32_t off[kPubMax + 1];
  int n;
  uint32_t tag;
  uint32_t* dst;
};

// By one wavefront.  After the items, dst[0] receives `tag`, stored only once
// every word is visible at system scope: a host that reads the tag it expects,
// then the words, reads this call's values.  The word is never used for
// anything else, so an old value there is an older tag.  Items may have been
// written by this wavefront before the call.  One wavefront, because each that
// takes part in the fences pays for them: a scan by sixteen took 12 to 15 us with
// them and takes 8 to 9.
__device__ __forceinline__ void publish_items(const PubArgs& a) {
  const uint32_t lane = threadIdx.x;
  __threadfence();
  for (int k = 0; k < a.n; ++k) {
    const uint32_t* src = a.src[k];
    const uint32_t o = a.off[k], len = a.off[k + 1] - o;
    for (uint32_t w = lane; w < len; w += kWave)
      a.dst[1 + o + w] = __hip_atomic_load(src + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __threadfence_system();
  if (lane == 0) __hip_atomic_store(a.dst, a.tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(kWave) k_publish(PubArgs a) { publish_items(a); }

// A thread's kScanItems consecutive counts (0 past n): two 16-byte loads where
// all of them exist and lie so, since one by one each load of a wavefront
// touched 16 lines for 64 counts (1.5 M counts: offsets 7.6 -> 4.4 us).
__device__ __forceinline__ void load_counts(const int* __restrict__ in, int n, long long base,
                                            int (&v)[kScanItems]) {
  if (base + kScanItems <= n && (reinterpret_cast<uintptr_t>(in) & 15) == 0) {
    const int4 a = *reinterpret_cast<const int4*>(in + base);
    const int4 b = *reinterpret_cast<const int4*>(in + base + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w;
    v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) v[k] = base + k < n ? in[base + k] : 0;
  }
}

// Block sums of the counts and, with bmax, block maxima (the scan then also
// delivers the largest count, which the callers need beside the total).
__global__ void __launch_bounds__(kBlock) k_scan_reduce(const int* __restrict__ in, int n,
                                                        long long* __restrict__ bsum,
                                                        int* __restrict__ bmax) {
  const long long base = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanItems;
  int v[kScanItems];
  load_counts(in, n, base, v);
  long long s = 0;
  int m = INT32_MIN;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    s += v[k];
    if (base + k < n) m = max(m, v[k]);
  }
  s = block_sum<kBlock>(s);
  if (threadIdx.x == 0) bsum[blockIdx.x] = s;
  if (bmax) {
    m = block_max<kBlock>(m);
    if (threadIdx.x == 0) bmax[blockIdx.x] = m;
  }
}

// Scan of the block sums; with mx, the largest block maximum is max-ed into
// *mx (as k_max_int does).  What pub names is published from here, so the host
// goes on while the offsets are still being written.
__global__ void __launch_bounds__(kBlock) k_scan_top(long long* __restrict__ bsum, int nb,
                                                     long long* __restrict__ total,
                                                     const int* __restrict__ bmax,
                                                     int* __restrict__ mx, PubArgs pub) {
  long long carry = 0;
  for (int base = 0; base < nb; base += kBlock) {
    int i = base + threadIdx.x;
    long long v = i < nb ? bsum[i] : 0;
    long long t;
    long long ex = block_excl_scan(v, &t);
    if (i < nb) bsum[i] = carry + ex;
    carry += t;
  }
  if (threadIdx.x == 0) *total = carry;
  if (mx) {
    int m = INT32_MIN;
    for (int i = threadIdx.x; i < nb; i += kBlock) m = max(m, bmax[i]);
    m = block_max<kBlock>(m);
    if (threadIdx.x == 0) atomicMax(mx, m);
  }
  if (pub.dst && threadIdx.x < kWave) publish_items(pub);
}

__global__ void __launch_bounds__(kBlock) k_scan_down(const int* __restrict__ in, int n,
                                                      const long long* __restrict__ boff,
                                                      const long long* __restrict__ total,
                                                      int* __restrict__ out) {
  const long long base = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanItems;
  int v[kScanItems];
  load_counts(in, n, base, v);
  long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += v[k];
  long long t;
  long long run = block_excl_scan(s, &t) + boff[blockIdx.x];
  int o[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    o[k] = (int)run;
    run += v[k];
  }
  if (base + kScanItems <= n && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    *reinterpret_cast<int4*>(out + base) = make_int4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<int4*>(out + base + 4) = make_int4(o[4], o[5], o[6], o[7]);
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
      if (base + k < n) out[base + k] = o[k];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = (int)*total;
}

// Inclusive scan of 32-bit values over a wavefront in DPP shifts: within rows
// of 16 lanes, then across them.
__device__ __forceinline__ int wave_incl_scan32(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Exclusive scan of n <= kSmallScan counts by one block of kSmallBlock
// threads, the counts in registers: every wavefront scans its 64 counts of each
// run of kSmallBlock, one wavefront scans the wavefronts' sums.  out[0..n],
// *total.  The total is summed in 64 bits; offsets are 32-bit, exact whenever
// the total is (a larger one is an error of the caller's).  One compute unit's
// loads and two barriers bound it: 0.6 to 13.8 k counts take 5 to 6 us, 8 to 9 with
// what it publishes.
constexpr int kSmallBlock = 1024;
constexpr int kSmallItems = 15;
constexpr int kSmallScan = kSmallBlock * kSmallItems;

__global__ void __launch_bounds__(kSmallBlock) k_scan_small(const int* __restrict__ in, int n,
                                                            int* __restrict__ out,
                                                            long long* __restrict__ total,
                                                            int* __restrict__ mx, PubArgs pub) {
  constexpr int kWaves = kSmallBlock / kWave;
  __shared__ int wsum[kSmallItems * kWaves];  // in scan order; 240 <= 4 a lane
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  int m = INT32_MIN;
  long long sum = 0;
  int item[kSmallItems], inc[kSmallItems];
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    const int i = threadIdx.x + k * kSmallBlock;
    item[k] = n > 0 ? in[i < n ? i : 0] : 0;
  }
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    const int i = threadIdx.x + k * kSmallBlock;
    if (i < n) m = max(m, item[k]);
    else item[k] = 0;
    sum += item[k];
    inc[k] = wave_incl_scan32(item[k]);
    if (lane == kWave - 1) wsum[k * kWaves + w] = inc[k];
  }
  if (mx) {  // the largest count, max-ed into *mx as k_max_int does
    m = block_max<kSmallBlock>(m);
    if (threadIdx.x == 0) atomicMax(mx, m);
  }
  sum = block_sum<kSmallBlock>(sum);  // also the barrier before wsum is read
  if (w == 0) {
    int v[4], s4 = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = 4 * lane + u;
      v[u] = q < kSmallItems * kWaves ? wsum[q] : 0;
      s4 += v[u];
    }
    int run = wave_incl_scan32(s4) - s4;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = 4 * lane + u;
      if (q < kSmallItems * kWaves) wsum[q] = run;
      run += v[u];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    const int i = threadIdx.x + k * kSmallBlock;
    const int off = wsum[k * kWaves + w] + inc[k] - item[k];
    if (i < n) out[i] = off;
  }
  if (threadIdx.x == 0) {
    out[n] = (int)sum;
    *total = sum;
  }
  if (pub.dst && threadIdx.x < kWave) publish_items(pub);
}

__global__ void __launch_bounds__(kBlock) k_max_int(const int* __restrict__ in, int n,
                                                    int* __restrict__ out) {
  int m = INT32_MIN;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    m = max(m, in[i]);
  m = block_max<kBlock>(m);
  if (threadIdx.x == 0) atomicMax(out, m);
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_fill(T* __restrict__ p, T v, long long n) {
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (long long)gridDim.x * kBlock)
    p[i] = v;
}

}  // namespace

int scan_blocks(int n) {
  int nb = (int)((n + (int64_t)kScanTile - 1) / kScanTile);
  return nb < 1 ? 1 : nb;
}

// Where the scan of n counts through a slot leaves its total: after the block
// sums, before (with max_out) the block maxima as ints.
static long long* scan_total(ppe_solver* s, int n, int slot, const int* max_out) {
  const int nb = n <= kSmallScan ? 1 : scan_blocks(n);
  return s->tmp_l[slot].get<long long>(nb + 1 + (max_out ? (nb + 1) / 2 : 0)) + nb;
}

static PubArgs pub_args(ppe_solver* s, const ReadItem* items, int n, size_t at) {
  if (n > kPubMax) throw Error(PPE_ERR_INTERNAL, "too many read-back items in one call");
  PubArgs a{};
  a.n = n;
  uint32_t off = 0;
  for (int k = 0; k < n; ++k) {
    if (items[k].bytes % 4 != 0) throw Error(PPE_ERR_INTERNAL, "read-back size not a word multiple");
    a.src[k] = static_cast<const uint32_t*>(items[k].dev);
    a.off[k] = off;
    off += (uint32_t)(items[k].bytes / 4);
  }
  a.off[n] = off;
  ensure_box(s, at + off + 1);
  a.tag = ++s->box_tag;
  a.dst = s->box_d + at;
  return a;
}

static void read_items(ppe_solver* s, const Published& pub, const std::vector<ReadItem>& items) {
  const uint32_t* h = published_words(s, pub);
  for (const auto& it : items) {
    std::memcpy(it.host, h, it.bytes);
    h += it.bytes / 4;
  }
}

static long long* scan_launch(ppe_solver* s, const int* in, int* out, int n, int slot, int* max_out,
                              const PubArgs& pub) {
  if (n < 0) throw Error(PPE_ERR_INTERNAL, "negative scan length");
  long long* total = scan_total(s, n, slot, max_out);
  if (n <= kSmallScan) {
    hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(kSmallBlock), 0, s->stream, in, n, out, total,
                       max_out, pub);
    PPE_LAUNCH_CHECK();
    return total;
  }
  const int nb = scan_blocks(n);
  long long* bsum = total - nb;
  int* bmax = max_out ? reinterpret_cast<int*>(total + 1) : nullptr;
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kBlock), 0, s->stream, in, n, bsum, bmax);
  PPE_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlock), 0, s->stream, bsum, nb, total,
                     (const int*)bmax, max_out, pub);
  PPE_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kBlock), 0, s->stream, in, n, bsum, total, out);
  PPE_LAUNCH_CHECK();
  return total;
}

long long* exclusive_scan_async(ppe_solver* s, const int* in, int* out, int n, int slot,
                                int* max_out) {
  return scan_launch(s, in, out, n, slot, max_out, PubArgs{});
}

long long exclusive_scan_read(ppe_solver* s, const int* in, int* out, int n, int* max_out,
                              std::initializer_list<ReadItem> more) {
  long long t = 0;
  std::vector<ReadItem> all{ReadItem{scan_total(s, n, 0, max_out), sizeof(long long), &t}};
  all.insert(all.end(), more);
  const PubArgs pub = pub_args(s, all.data(), (int)all.size(), kBoxRead);
  scan_launch(s, in, out, n, 0, max_out, pub);
  read_items(s, Published{s->box_h + kBoxRead, pub.tag}, all);
  return t;
}

int64_t exclusive_scan(ppe_solver* s, const int* in, int* out, int n) {
  const long long t = exclusive_scan_read(s, in, out, n, nullptr, {});
  if (t > INT32_MAX) throw Error(PPE_ERR_INTERNAL, "scan total exceeds int32 range");
  return t;
}

void max_int_async(ppe_solver* s, const int* in, int n, int* out, bool init) {
  if (init) fill_int(s, out, INT32_MIN, 1);
  int g = grid_for(n);
  if (g > 1024) g = 1024;
  hipLaunchKernelGGL(k_max_int, dim3(g), dim3(kBlock), 0, s->stream, in, n, out);
  PPE_LAUNCH_CHECK();
}

int reduce_max_int(ppe_solver* s, const int* in, int n) {
  int* out = s->tmp_i[3].get<int>(1);
  fill_int(s, out, INT32_MIN, 1);
  int g = grid_for(n);
  if (g > 1024) g = 1024;
  hipLaunchKernelGGL(k_max_int, dim3(g), dim3(kBlock), 0, s->stream, in, n, out);
  PPE_LAUNCH_CHECK();
  return read_scalar(s, out);
}

void ensure_box(ppe_solver* s, size_t words) {
  if (words <= s->box_words) return;
  size_t cap = s->box_words ? s->box_words : 4096;
  while (cap < words) cap *= 2;
  if (s->box_h) {
    // kernels in flight may still write the old box
    PPE_HIP(hipStreamSynchronize(s->stream));
    PPE_HIP(hipHostFree(s->box_h));
    s->box_h = s->box_d = nullptr;
    s->box_words = 0;
  }
  void* h = nullptr;
  PPE_HIP(hipHostMalloc(&h, cap * sizeof(uint32_t), hipHostMallocMapped | hipHostMallocCoherent));
  std::memset(h, 0, cap * sizeof(uint32_t));  // no tag: they count from 1
  void* d = nullptr;
  PPE_HIP(hipHostGetDevicePointer(&d, h, 0));
  s->box_h = static_cast<uint32_t*>(h);
  s->box_d = static_cast<uint32_t*>(d);
  s->box_words = cap;
}

Published publish(ppe_solver* s, const ReadItem* items, int n, size_t at) {
  const PubArgs a = pub_args(s, items, n, at);
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(kWave), 0, s->stream, a);
  PPE_LAUNCH_CHECK();
  return Published{s->box_h + at, a.tag};
}

// The tag is watched rather than the stream: the words are there once the tag
// is, some microseconds before a wait for the stream would return, and neither a
// signal nor an event has to be queued behind the kernel (16^3: assembly 502 ->
// 468 us, solve 477 -> 466, and 575 + 499 in processes whose stream waits sleep;
// a 64^3 projection 2.54, or 2.73, -> 2.46 ms).  After
// kTagSpin the stream is waited for, which also reports a failed kernel.
constexpr std::chrono::microseconds kTagSpin(2000);

const uint32_t* published_words(ppe_solver* s, const Published& p) {
  auto tag_now = [&]() {
    return __atomic_load_n(p.box, __ATOMIC_ACQUIRE);
  };
  const auto until = std::chrono::steady_clock::now() + kTagSpin;
  for (int k = 0; tag_now() != p.tag; ++k) {
    __builtin_ia32_pause();
    if (k % 64 == 63 && std::chrono::steady_clock::now() > until) {
      PPE_HIP(hipStreamSynchronize(s->stream));
      if (tag_now() != p.tag)
        throw Error(PPE_ERR_INTERNAL, "read-back values not visible to the host");
      break;
    }
  }
  return p.box + 1;
}

void read_back(ppe_solver* s, std::initializer_list<ReadItem> items) {
  const std::vector<ReadItem> all(items);
  read_items(s, publish(s, all.data(), (int)all.size(), kBoxRead), all);
}

void fill_int(ppe_solver* s, int* p, int v, int64_t n) {
  if (n <= 0) return;
  int g = grid_for(n);
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_fill<int>, dim3(g), dim3(kBlock), 0, s->stream, p, v, (long long)n);
  PPE_LAUNCH_CHECK();
}

void fill_double(ppe_solver* s, double* p, double v, int64_t n) {
  if (n <= 0) return;
  int g = grid_for(n);
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_fill<double>, dim3(g), dim3(kBlock), 0, s->stream, p, v, (long long)n);
  PPE_LAUNCH_CHECK();
}

}  // namespace ppe
