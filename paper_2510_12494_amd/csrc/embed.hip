// Sparse SGD step on the embedding tables of the categorical bottoms on
// gfx950 (the gather of the looked-up rows is part of the chain kernels'
// input stage).
//
// The sparse step (Eq. 2 restricted to the table rows a batch touches) sums,
// for every touched table row, the gradient rows of all samples that looked
// it up, and applies SGD once per touched row.
//
// Work split: no two wavefronts ever write the same table row.  The ids of a
// field are dealt to kParts = 64 parts by a mix of their bits (mix_id: a
// permutation of the 19-bit ids; its upper 6 bits are the part); a workgroup
// takes four parts of one field, a wavefront one of them.  Per pass of up to
// 8192 samples
//   1. the workgroup reads the field's ids (a field-major copy the gather
//      wrote) once and places the (rest of the mixed id, row) keys of its
//      four parts into LDS, part by part, in a fixed order (a scan of
//      per-thread counts);
//   2. a frequent id is found in a sample of 64 of the part's keys (one that
//      holds at least kHotSample of them), taken out of the list and summed
//      in list order, kQueue rows per wavefront in flight, whatever its value
//      is: with Zipf-like fields the first ids carry a large share of the
//      samples (exponent 1.1 over 100k ids: 13 %, 6 %, 4 %, ..), and sorting
//      them would cost more than reading them.  Lists of more than kShareMin
//      keys are gone through by all four wavefronts, a quarter each;
// then each wavefront works on its part alone, without a barrier:
//   3. the other keys are sorted (bitonic network in registers up to 1024
//      keys, in LDS beyond), by id, then by sample;
//   4. segmented sums per id over the sorted keys, 128 positions at a time:
//      16 lane groups (4 lanes: the row's 4-column chunks) take 8
//      consecutive positions each, their gradient and table rows loaded
//      together, a scan over the groups combines the segments that cross
//      them, and the updated table row is stored where its segment ends.
// The order of every sum depends only on the ids, so two runs give bitwise
// the same tables.
//
// Bound by latency (dependent id, key, gradient and table reads), so many
// small independent wavefronts, and no long work for one of them.  us per
// tick of 13 fields per party, 8192 samples, one stream: a workgroup per part
// of 16 and per id 0 .. 15 with its barriers / a wavefront per part of id mod
// 64 and per frequent id / this one: 100,000 ids 36 / 28 / 27; one id 39 / 65 /
// 33; two 26 / 44 / 22; ten 34 / 37 / 27; multiples of 64 147 / 1059 / 27 (all
// in one part, where one wavefront sorted 8192 keys in LDS).  us a launch of
// 30,000 samples of 6 fields, 8-wide rows (four passes), the first / this one:
// 1000 ids 63 / 56, two 52 / 57, one 58 / 67 (the ticks 2389 / 2053, 2198 /
// 2088 and 2276 / 2226 us an epoch of 12).
#include <algorithm>

#include "device.h"
#include "kernels.h"

namespace vfl {
namespace {
using namespace dev;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kRowBits = 13;
constexpr int kPass = 1 << kRowBits;           // samples per pass
constexpr uint32_t kRowMask = kPass - 1;
constexpr int kRowsPerThread = kPass / kThreads;     // rows a thread tests per pass
constexpr int kParts = 64;                     // id parts per field
constexpr int kBlocksPerField = kParts / kWaves;
constexpr int kShareMin = 512;                 // keys above which the workgroup goes through a list together
constexpr int kHotMin = 128;                   // keys from which frequent ids are looked for
constexpr int kHotSample = 8;                  // of 64 sampled keys: such an id is taken out
constexpr int kQueue = 128;                    // rows of a frequent id summed together
constexpr int kStage = 128;                    // sorted positions per stage
constexpr int kGroups = 16;                    // 4-lane groups per wavefront
constexpr int kSpan = kStage / kGroups;        // positions per group
constexpr uint32_t kNone = 0xFFFFFFFFu;

// The part of an id, and what tells it from the part's other ids: a
// permutation of the 19-bit ids, by an exclusive or with their upper bits
// and a multiplication with 2^19 over the golden ratio (odd), which deals
// out consecutive ids, multiples of a power of two (id mod 64 put all of them
// in one part) and of other strides evenly.
constexpr int kIdBits = 19, kSubBits = kIdBits - 6;
constexpr uint32_t kIdMask = (1u << kIdBits) - 1, kSubMask = (1u << kSubBits) - 1;
constexpr uint32_t kMul = 324027u;
constexpr uint32_t inverse(uint32_t m) {
  uint32_t x = m;                              // correct to 3 bits; each step doubles them
  for (int i = 0; i < 4; ++i) x *= 2u - m * x;
  return x & kIdMask;
}
constexpr uint32_t kMulInv = inverse(kMul);
static_assert(((kMul * kMulInv) & kIdMask) == 1u && kParts == 1 << 6 && kSubBits + kRowBits <= 32 && 2 * 10 >= kIdBits,
              "the mix is not a permutation");
__device__ __forceinline__ uint32_t mix_id(uint32_t id) { return __umul24(id ^ (id >> 10), kMul) & kIdMask; }
__device__ __forceinline__ uint32_t unmix_id(uint32_t h) {
  const uint32_t y = __umul24(h, kMulInv) & kIdMask;
  return y ^ (y >> 10);
}

// keeps the LDS accesses of a wavefront's lanes in program order (the
// hardware does; this holds the compiler to it)
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ f32x4 shfl_up4(const f32x4& v, int d) {
  f32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = __shfl_up(v[e], d, 64);
  return r;
}
__device__ __forceinline__ f32x4 shfl4(const f32x4& v, int lane) {
  f32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = __shfl(v[e], lane, 64);
  return r;
}
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Ascending bitonic sort of a[0, n), n <= 64 * KPT, by one wavefront: lane l
// holds the slots [l * KPT, l * KPT + KPT) in registers (padded with kNone).
template <int KPT>
__device__ __forceinline__ void sort_regs(uint32_t* a, int n) {
  constexpr int N = 64 * KPT;
  const int t = threadIdx.x & 63;
  uint32_t x[KPT];
#pragma unroll
  for (int e = 0; e < KPT; ++e) x[e] = t * KPT + e < n ? a[t * KPT + e] : kNone;
#pragma unroll 1
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll 1
    for (int h = k >> 1; h >= KPT; h >>= 1) {
      // bit k of a slot index lies in t * KPT (k > h >= KPT)
      const bool asc = ((t * KPT) & k) == 0, lower = ((t * KPT) & h) == 0;
      const bool keep_min = asc == lower;
      const int m = h / KPT;
#pragma unroll
      for (int e = 0; e < KPT; ++e) {
        const uint32_t o = (uint32_t)__shfl_xor((int)x[e], m, 64);
        x[e] = keep_min ? min(x[e], o) : max(x[e], o);
      }
    }
    // distances below KPT: inside the lane
#pragma unroll
    for (int h = KPT / 2; h >= 1; h >>= 1) {
      if (h >= k) continue;
#pragma unroll
      for (int e = 0; e < KPT; ++e) {
        if (e & h) continue;
        const bool asc = ((t * KPT + e) & k) == 0;
        const uint32_t lo = min(x[e], x[e + h]), hi = max(x[e], x[e + h]);
        x[e] = asc ? lo : hi;
        x[e + h] = asc ? hi : lo;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < KPT; ++e)
    if (t * KPT + e < n) a[t * KPT + e] = x[e];
  lds_order();
}

// the same in LDS, any n (slots past n count as kNone: an exchange with
// one never moves a key there, because the network's last half-cleaner
// directions leave the largest at the end)
__device__ __forceinline__ void sort_lds(uint32_t* a, int n) {
  const int t = threadIdx.x & 63;
  int N = 64;
  while (N < n) N <<= 1;
  // the bitonic network with every comparison ascending (the first step of
  // each merge compares mirrored slots), so that slots past n stay the
  // largest and need no storage
  for (int k = 2; k <= N; k <<= 1) {
    for (int h = k >> 1; h >= 1; h >>= 1) {
      for (int p = t; p < N / 2; p += 64) {
        const int lo = (p / h) * 2 * h + p % h;
        const int hi = h == k >> 1 ? (lo / k) * k + k - 1 - lo % k : lo + h;
        if (hi < n) {
          const uint32_t x = a[lo], y = a[hi];
          if (x > y) { a[lo] = y; a[hi] = x; }
        }
      }
      lds_order();
    }
  }
}

__global__ __launch_bounds__(kThreads, 3) void k_embed_sgd(ScatterJob j) {
  __shared__ uint32_t keys[kPass];
  __shared__ uint16_t queue[kWaves][kQueue + 64];
  __shared__ uint32_t wcnt[kWaves][2];
  __shared__ f32x4 psum[2][kWaves][4];          // a shared list's wavefront sums (two iterations)
  __shared__ int plen[kWaves];                  // and how many keys each has left in its quarter
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f = blockIdx.x / kBlocksPerField, quad = blockIdx.x % kBlocksPerField;
  int R = j.R;
  float scale = j.scale;
  if (j.tr.src) {
    const TickArgs ta = tick_args(j.tr);
    R = ta.rows;
    scale = ta.scale;
  }
  const int EC = j.E / 4;                       // 4-column chunks per table row
  const VFL_GLOBAL int32_t* ids = glb(j.idt) + (int64_t)f * j.ldi;
  const int grp = lane >> 2, ch = lane & 3;     // lane group, chunk
  const int cc = min(ch, EC - 1);               // lanes past E repeat its last chunk (never stored)
  // a pass's gradient rows and the field's table through uniform bases with
  // 32-bit byte offsets (8192 rows of at most 64K floats; 2^19 rows of 64
  // bytes), so that a load needs one address register
  const uint32_t part = (uint32_t)(kWaves * quad + wave);
  const VFL_GLOBAL char* Gb = glb((const char*)j.G) + (int64_t)f * EC * 16;
  VFL_GLOBAL char* Tb = glb((char*)(j.T + (int64_t)f * j.V * j.E));
  const uint32_t ldg = (uint32_t)j.ldg * 4u, row_bytes = 16u * (uint32_t)EC, lo = 16u * (uint32_t)cc;
  auto row_at = [&](uint32_t p, uint32_t sub) { // this lane's chunk of the table row of part p's id
    return (VFL_GLOBAL f32x4*)(Tb + (uint32_t)(unmix_id(p << kSubBits | sub) * row_bytes + lo));
  };
  auto table_row = [&](uint32_t sub) { return row_at(part, sub); };
  uint16_t* q = queue[wave];

  for (int c0 = 0; c0 < R; c0 += kPass) {
    const int n = min(kPass, R - c0);
    // 1. every thread tests kPass / kThreads rows (strided, so each load
    // instruction of a wavefront is contiguous) and counts those of each of
    // the workgroup's parts, in a byte each
    uint32_t idv[kRowsPerThread];             // mixed
    auto sub_part = [&](int i) {              // the row's part here, >= kWaves: not in this workgroup
      return (idv[i] >> kSubBits) - (uint32_t)(kWaves * quad);
    };
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) idv[i] = (uint32_t)ids[c0 + min(i * kThreads + tid, n - 1)];
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) idv[i] = mix_id(idv[i]);
    uint32_t count = 0u;
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) {
      const uint32_t x = sub_part(i);
      count += x < (uint32_t)kWaves && i * kThreads + tid < n ? 1u << (8 * x) : 0u;
    }
    // the counts of parts 0, 1 and 2, 3 as 16-bit halves (at most kPass
    // together): scans over the lanes, then over the wavefronts
    uint32_t cnt[2], incl[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t x = count >> (16 * h);
      cnt[h] = (x & 0xffu) | (x & 0xff00u) << 8;
      incl[h] = cnt[h];
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl[h], d, 64);
        if (lane >= d) incl[h] += v;
      }
    if (lane == 63) { wcnt[wave][0] = incl[0]; wcnt[wave][1] = incl[1]; }
    __syncthreads();
    uint32_t before[2] = {0u, 0u}, total[2] = {0u, 0u};
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t x = wcnt[w][h];
        before[h] += w < wave ? x : 0u;
        total[h] += x;
      }
    int base[kWaves + 1];
    uint32_t pos[2];                          // of the thread's next key, packed like the counts
    base[0] = 0;
#pragma unroll
    for (int s = 0; s < kWaves; ++s) base[s + 1] = base[s] + (int)((total[s >> 1] >> (16 * (s & 1))) & 0xffffu);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      pos[h] = before[h] + incl[h] - cnt[h] + ((uint32_t)base[2 * h] | (uint32_t)base[2 * h + 1] << 16);
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) {
      const uint32_t x = sub_part(i);
      if (x < (uint32_t)kWaves && i * kThreads + tid < n) {
        const uint32_t sh = 16 * (x & 1), p = x & 2 ? pos[1] : pos[0];
        keys[(p >> sh) & 0xffffu] = ((idv[i] & kSubMask) << kRowBits) | (uint32_t)(i * kThreads + tid);
        pos[0] += x & 2 ? 0u : 1u << sh;
        pos[1] += x & 2 ? 1u << sh : 0u;
      }
    }
    __syncthreads();
    const VFL_GLOBAL char* Gp = Gb + (int64_t)c0 * ldg;
    auto grad_row = [&](uint32_t row) { return *(const VFL_GLOBAL f32x4*)(Gp + (uint32_t)(row * ldg + lo)); };

    // 2. frequent ids.  The one most of the 64 lanes hold (sid) and how many
    // do (at least 8 leave a list each time, so the loops below end).
    auto frequent = [&](uint32_t sid, uint32_t& id) {
      int same = 0;
#pragma unroll 8
      for (int l = 0; l < 64; ++l) same += sid == (uint32_t)__builtin_amdgcn_readlane((int)sid, l) ? 1 : 0;
      int best = same << 6 | lane;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) best = max(best, __shfl_xor(best, d, 64));
      best = __builtin_amdgcn_readfirstlane(best);
      id = (uint32_t)__builtin_amdgcn_readlane((int)sid, best & 63);
      return best >> 6;
    };
    // takes the keys of id `hot` out of list[0, n), n > 0, and sums their
    // gradient rows; returns the keys left, sum in the lanes of group 0.
    // one: all sampled keys are of that id
    auto take_out = [&](uint32_t* list, int n, uint32_t hot, bool one, f32x4& sum) {
      sum = f32x4{0.f, 0.f, 0.f, 0.f};
      // rows q[0, m) (m <= kQueue) are loaded together, a lane group every
      // 16th, and added, in order, once the next ones are found
      f32x4 v[kQueue / kGroups];
      int loaded = 0;
      auto add_loaded = [&] {
        if (loaded == kQueue) {
#pragma unroll
          for (int u = 0; u < kQueue / kGroups; ++u) sum += v[u];
          return;
        }
#pragma unroll
        for (int u = 0; u < kQueue / kGroups; ++u)
          if (u * kGroups + grp < loaded) sum += v[u];
      };
      auto load_rows = [&](int m) {
#pragma unroll
        for (int u = 0; u < kQueue / kGroups; ++u) v[u] = grad_row(q[min(u * kGroups + grp, m - 1)]);
        loaded = m;
      };
      int rest = 0, qn = 0, i0 = 0;
      // While the next kQueue keys are all of this id (a field of few ids has
      // most of them in parts of their own), the rows are read straight from
      // the list, the same ones together as through the queue: a turn of the
      // queue is a chain of LDS reads and writes that takes as long as the
      // gradient rows (one id, 30,000 samples of 6 fields: 83 us a launch
      // through the queue, 67 so)
      for (; one && i0 + kQueue <= n; i0 += kQueue) {
        uint32_t k[kQueue / kGroups], other = 0u;
#pragma unroll
        for (int u = 0; u < kQueue / kGroups; ++u) k[u] = list[i0 + u * kGroups + grp];
#pragma unroll
        for (int u = 0; u < kQueue / kGroups; ++u) other |= (k[u] >> kRowBits) ^ hot;
        if (__ballot(other != 0u)) break;
        add_loaded();
#pragma unroll
        for (int u = 0; u < kQueue / kGroups; ++u) v[u] = grad_row(k[u] & kRowMask);
        loaded = kQueue;
      }
      for (; i0 < n; i0 += 64) {
        const bool in = i0 + lane < n;
        const uint32_t key = list[min(i0 + lane, n - 1)];
        const bool is = in && (key >> kRowBits) == hot;
        const uint64_t bh = __ballot(is), br = __ballot(in && !is);
        lds_order();
        if (is) q[qn + lanes_below(bh)] = (uint16_t)(key & kRowMask);
        else if (in) list[rest + lanes_below(br)] = key;   // at or below i0 + lane: read already
        rest += __builtin_popcountll(br);
        qn += __builtin_popcountll(bh);
        lds_order();
        if (qn >= kQueue) {
          add_loaded();
          load_rows(kQueue);
          const uint16_t left = q[kQueue + lane];
          lds_order();
          if (lane < qn - kQueue) q[lane] = left;
          qn -= kQueue;
          lds_order();
        }
      }
      add_loaded();
      if (qn > 0) {
        load_rows(qn);
        add_loaded();
      }
      // the 16 groups (lanes 4 apart), a fixed tree
#pragma unroll
      for (int d = 32; d >= 4; d >>= 1) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __shfl_down(sum[e], d, 64);
        sum += o;
      }
      return rest;
    };

    int b0 = base[0], np = base[1] - base[0];
#pragma unroll
    for (int s = 1; s < kWaves; ++s)
      if (wave == s) { b0 = base[s]; np = base[s + 1] - base[s]; }
    b0 = __builtin_amdgcn_readfirstlane(b0);
    np = __builtin_amdgcn_readfirstlane(np);
    uint32_t* list = keys + b0;

    // long lists together, one after the other: wavefront w goes through the
    // w-th quarter; the owner adds the four sums in wavefront order.  Every
    // wavefront takes the same turns (the counts and samples are the same
    // for all, and no list changes between a sample and the barrier after it)
#pragma unroll 1
    for (int s = 0; s < kWaves; ++s) {
      int sb = base[0], sn = base[1] - base[0];
#pragma unroll
      for (int u = 1; u < kWaves; ++u)
        if (s == u) { sb = base[u]; sn = base[u + 1] - base[u]; }
      sb = __builtin_amdgcn_readfirstlane(sb);
      sn = __builtin_amdgcn_readfirstlane(sn);
      if (sn <= kShareMin) continue;
      int at[kWaves], len[kWaves];              // the quarters
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        at[w] = sb + sn * w / kWaves;
        len[w] = sb + sn * (w + 1) / kWaves - at[w];
      }
#pragma unroll 1
      for (int it = 0; sn > kShareMin; it ^= 1) {
        const int x = (lane * sn) >> 6;
        int pos = at[0] + x, end = len[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
          if (x >= end) pos = at[w] + x - end;
          end += len[w];
        }
        uint32_t hot;
        const int share = frequent(keys[pos] >> kRowBits, hot);
        __syncthreads();
        if (share < kHotSample) break;
        int a = at[0], m = len[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w)
          if (wave == w) { a = at[w]; m = len[w]; }
        f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
        if (m > 0) m = take_out(keys + a, m, hot, share == 64, sum);
        if (lane < 4) psum[it][wave][lane] = sum;
        if (lane == 0) plen[wave] = m;
        __syncthreads();
        sn = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          len[w] = __builtin_amdgcn_readfirstlane(plen[w]);
          sn += len[w];
        }
        if (wave == s && lane < EC) {
          f32x4 t = psum[it][0][lane];
#pragma unroll
          for (int w = 1; w < kWaves; ++w) t += psum[it][w][lane];
          VFL_GLOBAL f32x4* row = row_at(part, hot);   // (lane = chunk here)
          *row = *row - scale * t;
        }
      }
      if (wave == s) {
        // what is left of the quarters, end to end (never above its place)
        int to = at[0] + len[0];
#pragma unroll 1
        for (int w = 1; w < kWaves; ++w) {
          int from = at[1], m = len[1];
#pragma unroll
          for (int u = 2; u < kWaves; ++u)
            if (w == u) { from = at[u]; m = len[u]; }
          for (int i0 = 0; i0 < m; i0 += 64) {
            const uint32_t key = keys[from + min(i0 + lane, m - 1)];
            lds_order();
            if (i0 + lane < m) keys[to + i0 + lane] = key;
            lds_order();
          }
          to += m;
        }
        np = to - b0;
      }
    }

    while (np > kHotMin) {
      uint32_t hot;
      const int share = frequent(list[(lane * np) >> 6] >> kRowBits, hot);
      if (share < kHotSample) break;
      f32x4 sum;
      np = take_out(list, np, hot, share == 64, sum);
      if (lane < EC) {
        VFL_GLOBAL f32x4* row = table_row(hot);   // (lane = chunk here)
        *row = *row - scale * sum;
      }
    }

    // 3. sort
    if (np <= 64) sort_regs<1>(list, np);
    else if (np <= 128) sort_regs<2>(list, np);
    else if (np <= 256) sort_regs<4>(list, np);
    else if (np <= 1024) sort_regs<16>(list, np);
    else sort_lds(list, np);

    // 4. segmented sums
    f32x4 carry = f32x4{0.f, 0.f, 0.f, 0.f};    // the open segment entering the stage
    for (int s0 = 0; s0 < np; s0 += kStage) {
      const int p0 = s0 + grp * kSpan;
      uint32_t id[kSpan + 2];                   // of positions p0 - 1 .. p0 + kSpan (kNone outside the list)
      f32x4 gv[kSpan], tv[kSpan];
#pragma unroll
      for (int u = 0; u < kSpan + 2; ++u) {
        const int p = p0 - 1 + u;
        const uint32_t key = list[min(max(p, 0), np - 1)];
        id[u] = p >= 0 && p < np ? key >> kRowBits : kNone;
        if (u >= 1 && u <= kSpan) {
          gv[u - 1] = grad_row(key & kRowMask);
          tv[u - 1] = *table_row(key >> kRowBits);
        }
      }
      // (a) the group's aggregate: F, whether a segment starts in it
      bool F = false;
      f32x4 V = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 1; u <= kSpan; ++u) {
        const f32x4 g = p0 + u - 1 < np ? gv[u - 1] : f32x4{0.f, 0.f, 0.f, 0.f};
        const bool head = id[u] != id[u - 1];
        V = head ? g : V + g;
        F = F || head;
      }
      // (b) inclusive scan over the groups (lanes 4 apart)
#pragma unroll
      for (int d = 1; d < kGroups; d <<= 1) {
        const f32x4 vu = shfl_up4(V, 4 * d);
        const bool fu = __shfl_up((int)F, 4 * d, 64) != 0;
        if (grp >= d) {
          // (fu, vu) comes first
          V = F ? V : vu + V;
          F = F || fu;
        }
      }
      // what enters the group: the stage's carry, then the earlier groups
      const f32x4 ve = shfl_up4(V, 4);
      const bool fe = __shfl_up((int)F, 4, 64) != 0;
      f32x4 run = grp == 0 ? carry : (fe ? ve : carry + ve);
      // (c) walk again; update where a segment ends
#pragma unroll
      for (int u = 1; u <= kSpan; ++u) {
        run = id[u] != id[u - 1] ? gv[u - 1] : run + gv[u - 1];
        if (p0 + u - 1 < np && id[u] != id[u + 1] && ch < EC)
          *table_row(id[u]) = tv[u - 1] - scale * run;
      }
      // the open segment after the stage (a full one: all positions valid)
      const f32x4 vl = shfl4(V, 60 + ch);
      const bool fl = __shfl((int)F, 60 + ch, 64) != 0;
      carry = fl ? vl : carry + vl;
    }
    __syncthreads();   // the next pass refills the keys
  }
}

}  // namespace

hipError_t launch_scatter_sgd(const ScatterJob& j, hipStream_t st) {
  if (j.E > kMaxEmbDim || j.E % 4 || j.ldg % 4 || j.V > (1 << (32 - kRowBits))) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_embed_sgd, dim3(j.n_cat * kBlocksPerField), dim3(kThreads), 0, st, j);
  return hipGetLastError();
}

}  // namespace vfl
