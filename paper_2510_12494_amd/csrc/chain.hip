// Fused row-block kernels of the split-learning step on gfx950 (k_fwd,
// k_active, k_bwd; see kernels.h for what each computes).
//
// A workgroup of 12 wavefronts owns BR = 16 * RT (RT = 1 .. 4) consecutive
// rows of the group and runs every layer of its chain on them, the
// activations and deltas staying in LDS.  Eight product wavefronts (two per
// SIMD) run the layers; each layer is one MFMA product
// out[BR x N] = in[BR x K] W^T: wavefront w takes the 16-column output tiles
// w, w+8, w+16, ... (two at a time), loads the weight fragments of its tiles
// straight from global memory (L2-resident: the workgroups of an XCD fetch
// the kernel's weights into its L2 at the start) two groups of two MFMA
// steps ahead, across layer boundaries, and the activation fragments from
// LDS; biases come from an LDS table filled at the start;
// v_mfma_f32_16x16x32_bf16 for bf16 operands, v_mfma_f32_16x16x4_f32 for
// float32, float32 accumulation.  The weight fragment is the MFMA's A
// operand, so a lane ends up with four consecutive output columns of one row.
//
// Four copy wavefronts write what a later kernel needs: while the product
// wavefronts run stage i + 1 (which reads stage i's output and writes
// another buffer) they copy stage i's output from LDS to HBM, and both meet
// at the barrier that ends the stage.  Stores and loads share one in-order
// counter on gfx950, so a wavefront that stores a copy (a loop whose store
// count the compiler does not know) waits for those writes before it may use
// weights loaded earlier; with the copies in wavefronts of their own the
// product wavefronts' waits are exact, and two load groups in flight are
// enough: the weights come from L2 within about 160 ns at 110 bytes per ns
// and CU, and groups of four steps gained nothing any more.  Measured on one
// stream against copies issued inside the next product: k_active 93 -> 82 us
// (private, 48 rows per block), 123 -> 109 (regression), 25.9 -> 22.9
// (dense_tabular); per tick 176 -> 166, 232 -> 217 and 46.2 -> 44.6 us.  Two
// copy wavefronts instead of four were 2 to 7 % slower per tick.
//
// LDS rows are padded to 16 bytes past a multiple of 128, so the 16 rows a
// fragment read touches fall in distinct banks.  After a layer, the tensors a
// later kernel needs go to HBM: row-major for messages, the RC layout for
// the operands of the weight gradients (transposed by the LDS reads of bf16
// chunks, element by element from float32 rows).
//
// Paper correspondence: bottom models f_A, f_B and the top model g of
// Section 3, the BCE loss of Eq. (1) and its gradient, the embedding and
// gradient messages of Section 4.1 with the per-row clip and Gaussian noise
// of the differential-privacy appendix, and the cut-layer backward through
// the clip of B's published embedding.
#include "device.h"
#include "kernels.h"

namespace vfl {
namespace {
using namespace dev;

template <typename T>
struct Ch {
  static constexpr int CE = 16 / (int)sizeof(T);   // elements per chunk = rows per RC chunk
  static constexpr int KS = 4 * CE;                // contraction depth of one MFMA step
};

// values of this launch, from the call or the tick record
struct Call {
  int rows, group, chk;
  int64_t row0;      // sample id of the group's row 0 (noise counter)
  int64_t in_off;    // dataset row offset of the inputs
  int32_t hdr[3];
};

__device__ __forceinline__ Call resolve(const ChainCall& c, const TickRef& tr) {
  Call k;
  if (tr.src) {
    const TickArgs ta = tick_args(tr);
    k.rows = ta.rows; k.group = ta.group; k.chk = ta.chk;
    k.row0 = ta.row0; k.in_off = ta.row0;
    k.hdr[0] = ta.hdr[0]; k.hdr[1] = ta.hdr[1]; k.hdr[2] = ta.hdr[2];
  } else {
    k.rows = c.rows; k.group = c.group; k.chk = c.chk;
    k.row0 = c.row0; k.in_off = 0;
    k.hdr[0] = c.hdr[0]; k.hdr[1] = c.hdr[1]; k.hdr[2] = c.hdr[2];
  }
  return k;
}

__device__ __forceinline__ char* lp(char* s, const LBuf& b, int r, int byte_col) {
  return s + b.off + r * b.pitch + byte_col;
}

// ------------------------------------------------------------ block product
constexpr int kNW = kChainWaves;    // product wavefronts per block (two per SIMD)
constexpr int kNT = 64 * kNW;        // product threads
constexpr int kBT = kNT + 64 * kChainCopyWaves;   // threads per block
// the copy threads, read from the launch: with the constant in its place the
// ticks of float32 chains with tables are 2.5 % longer (8192 samples of 13
// fields a party: 148 -> 152 us), the others the same
__device__ __forceinline__ int copy_threads() { return (int)blockDim.x - kNT; }
// Wavefronts per SIMD the register allocation has to allow: two blocks of
// 12 wavefronts on a CU (80 registers) up to `two` row tiles per block, else
// one (168).  At 80 registers k_bwd<bf16, 2> (82 without the bound) keeps two
// blocks on a CU (32768 rows of 500-1024-512-128: 47 -> 37 us) and
// k_active<bf16, 1> (86) leaves room for the other party's blocks
// (regression's tick 224 -> 217 us), each with one register spilled;
// k_active<., 2> would spill 35 (ctr's 55 -> 62 us).
constexpr int min_waves(int rt, int two) { return rt <= two ? 6 : 3; }
constexpr int kNTW = 2;              // 16-column output tiles per wavefront and pass
constexpr int PF = 2;                // MFMA steps per weight load group
constexpr int kLogitChunks = kMaxLogitCols / 256;   // 4-column chunks per lane in the logit stage

// Weight-fragment registers of a chain: two load groups of PF MFMA steps
// (ping-pong).  The groups of a chain's products form one stream: when a
// wavefront has issued the loads of a pass's last group, the next two loads
// it issues are groups 0 and 1 of the next pass or of the next product, so
// a product starts with both of its first groups already in flight.  A
// pass has an even number of groups (steps past K are skipped), so every
// pass starts in `wa`.
struct Pipe {
  u32x4 wa[PF][kNTW], wb[PF][kNTW];
};

// A pointer or value the compiler must keep in scalar registers (it is
// uniform, but derived through selects the compiler may place in vector
// registers, and a field loaded through a vector-register pointer is a
// vector-memory load whose wait drains every load in flight).
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const void*)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A job descriptor read through the constant address space: the jobs are
// written once, before any launch, so their fields may come through the
// scalar cache (scalar loads, counted apart from the vector loads in flight)
// even after the kernel's own stores.
#define VFL_CONST __attribute__((address_space(4)))
template <typename X>
__device__ __forceinline__ const VFL_CONST X& cst(const X& x) {
  return *(const VFL_CONST X*)&x;
}

// 16-column tiles of a product of N output columns (up to the MFMA depth)
template <typename T>
__device__ __forceinline__ int tiles_of(int N) {
  constexpr int KS = Ch<T>::KS;
  return (N + KS - 1) / KS * (KS / 16);
}

// The loads of two MFMA steps of a pass's tiles at p[] into d: one contiguous
// 1 KB fragment per tile and step of the packed operand, each a load with a
// uniform base, the lane's 32-bit offset and an immediate.  Loads are
// unconditional (a conditional load would make the compiler wait for it on
// the spot): tiles past the operand's last are clamped to it, and steps past
// K read what follows the tile (the next tile, or the slack behind the
// operand), never used.
template <int OFS>
__device__ __forceinline__ void wgroup(const VFL_GLOBAL char* const (&p)[kNTW], u32x4 (&d)[PF][kNTW]) {
  const uint32_t lo = (threadIdx.x & 63) * 16;
#pragma unroll
  for (int j = 0; j < kNTW; ++j)
#pragma unroll
    for (int q = 0; q < PF; ++q) d[q][j] = *(const VFL_GLOBAL u32x4*)((p[j] + (OFS + q) * 1024) + lo);
}

// the tiles of a wavefront's pass: wave + kNW * (kNTW * pass + j)
__device__ __forceinline__ void pass_tiles(int pass, int (&tile)[kNTW]) {
  const int wave = uniform((int)(threadIdx.x >> 6));
#pragma unroll
  for (int j = 0; j < kNTW; ++j) tile[j] = wave + kNW * (kNTW * pass + j);
}

// where the fragments of a pass's tiles start in the packed operand W
__device__ __forceinline__ void pass_bases(const void* W, int kst, int ntl, int pass, const VFL_GLOBAL char* (&p)[kNTW]) {
  int tile[kNTW];
  pass_tiles(pass, tile);
#pragma unroll
  for (int j = 0; j < kNTW; ++j)
    p[j] = glb((const char*)uniform_ptr((const char*)W + (uint64_t)(uint32_t)(min(tile[j], ntl - 1) * kst) * 1024));
}

// start the loads of groups 0 and 1 of L's first pass
template <typename T>
__device__ __forceinline__ void prefetch(const ChainLayer* L, Pipe& p) {
  const VFL_CONST ChainLayer& C = cst(*(const ChainLayer*)uniform_ptr(L));
  const VFL_GLOBAL char* base[kNTW];
  pass_bases(uniform_ptr(C.W), uniform(C.kst), uniform(tiles_of<T>(C.N)), 0, base);
  wgroup<0>(base, p.wa);
  wgroup<PF>(base, p.wb);
}

// Copy of a chain kernel's bias table into LDS (see BiasTab).
__device__ __forceinline__ void copy_bias(char* s, const BiasTab& b) {
  const VFL_GLOBAL f32x4* src = glb((const f32x4*)b.src);
  for (int i = threadIdx.x; i < b.n4; i += kNT) *(f32x4*)(s + b.off + 16 * i) = src[i];
}

// One 4-byte load per 128-byte line of this workgroup's slice of the
// kernel's weight ranges (slice = workgroup / 8 mod 32: the workgroups of
// one XCD share its L2), returned so that the caller can consume the values
// where it waits for its inputs anyway.  Up to 2 lines per thread and
// range; addresses are clamped into the range, so the loads are
// unconditional.
__device__ __forceinline__ uint32_t warm_l2(const WarmSet& w, const void* dummy) {
  const int slice = (blockIdx.x >> 3) & 31;
  uint32_t x = 0u;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int lines = w.lines[r];
    const int per = (lines + 31) >> 5;
    const int c0 = slice * per, c1 = min(lines, c0 + per);
    const VFL_GLOBAL uint32_t* base = glb((const uint32_t*)(lines > 0 ? w.p[r] : dummy));
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int c = c0 + (int)threadIdx.x + k * kNT;
      x ^= base[(int64_t)(c < c1 ? c : 0) * 32];
    }
  }
  return x;
}

// out[r][n] = epi(r, n, sum_k in[r][k] W[n][k], bias) for the block's rows:
// epi(lr, n, acc, bias) receives block rows lr + 16 t, output columns n .. n+3 (n a
// multiple of 4; bias[i] = bias[n + i] from the LDS table, zero without a
// bias or past N), for every row of the block and every column below N
// rounded up to the MFMA depth.  On entry p holds groups 0 and 1 of L's
// first pass; on return, groups 0 and 1 of `next`'s (nullable).
// Weight addresses are one uniform pointer per tile of the pass, advanced by
// the groups of an iteration, instead of a step and a tile clamped per load:
// about 45 scalar instructions less per refill.  500-1024-512-128 at 48 rows
// per block: k_fwd 136 -> 125 us, k_bwd 87 -> 84; ten 256-wide layers at 32
// rows: k_active 72 -> 70.6.
// FAST: load groups with both tiles and all steps run without a branch between
// their products (the same k_fwd 125 -> 120), which takes about 30 registers
// more.  For kernels at 48 rows per block alone: at 16 and 32 rows the
// registers are what lets two workgroups, or another kernel's, share the CU
// (k_active with it at 32 rows: 70.6 -> 68 us by itself, but the two-party
// tick with 65536-row tables 152 -> 156), and at 64 rows it spills.
template <typename T, int RT, bool FAST, typename Epi>
__device__ __forceinline__ void block_mm(const char* s, const ChainLayer& L, Pipe& p,
                                         const ChainLayer* next, Epi&& epi) {
  constexpr int NTW = kNTW;
  const int lane = threadIdx.x & 63;
  const int kc = lane >> 4, lr = lane & 15;
  const VFL_CONST ChainLayer& C = cst(L);
  const void* W = uniform_ptr(C.W);
  const int ntl = uniform(tiles_of<T>(C.N));
  const int nks = uniform(C.kst);
  const int ng = ((nks + PF - 1) / PF + 1) & ~1;
  const int bl = uniform(C.bl);
  LBuf in;
  in.off = C.in.off;
  in.pitch = C.in.pitch;
  const int npass = (ntl + kNW * NTW - 1) / (kNW * NTW);
  // the next product's operand; past the chain's end the loads repeat this
  // product's (never used: every refill issues the same loads, so the
  // compiler's wait counts stay exact)
  next = (const ChainLayer*)uniform_ptr(next);
  const VFL_CONST ChainLayer& CN = cst(next ? *next : L);
  const void* nW = uniform_ptr(CN.W);
  const int nkst = uniform(CN.kst), nntl = uniform(tiles_of<T>(CN.N));
  const char* xbase = s + in.off + lr * in.pitch + kc * 16;
#pragma unroll 1
  for (int pass = 0; pass < npass; ++pass) {
    int tile[NTW];
    pass_tiles(pass, tile);
    // this pass's fragments (groups 0 and 1 are in p), and where the loads
    // go once its groups are all issued: the next pass, or the next
    // product's first
    const bool more = pass + 1 < npass;
    const VFL_GLOBAL char* wp[NTW];
    const VFL_GLOBAL char* np[NTW];
    pass_bases(W, nks, ntl, pass, wp);
    pass_bases(more ? W : nW, more ? nks : nkst, more ? ntl : nntl, more ? pass + 1 : 0, np);
    f32x4 acc[NTW][RT];
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto xread = [&](int ks, u32x4 (&x)[RT]) {
#pragma unroll
      for (int t = 0; t < RT; ++t) x[t] = *(const u32x4*)(xbase + t * 16 * in.pitch + ks * 64);
    };
    auto mma = [&](int j, const u32x4& w, const u32x4 (&x)[RT]) {
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        if constexpr (sizeof(T) == 2) {
          acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x[t]), acc[j][t], 0, 0, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                __uint_as_float(w[e]), __uint_as_float(x[t][e]), acc[j][t], 0, 0, 0);
        }
      }
    };
    // two groups of an iteration, each refilled as soon as its products
    // have read it; the iteration's last loads are the next pass's when
    // this one has no further group
    const bool two = tile[NTW - 1] < ntl;
    auto group = [&](int k0, const u32x4 (&w)[PF][NTW]) {
      if constexpr (FAST) {
        if (two && k0 + PF <= nks) {
#pragma unroll
          for (int q = 0; q < PF; ++q) {
            u32x4 x[RT];
            xread(k0 + q, x);
#pragma unroll
            for (int j = 0; j < NTW; ++j) mma(j, w[q][j], x);
          }
          return;
        }
      }
#pragma unroll
      for (int q = 0; q < PF; ++q) {
        if (k0 + q >= nks || tile[0] >= ntl) continue;
        u32x4 x[RT];
        xread(k0 + q, x);
        mma(0, w[q][0], x);
        if (two) mma(1, w[q][1], x);
      }
    };
#pragma unroll 1
    for (int ks = 0; ks < ng * PF; ks += 2 * PF) {
      const bool last = ks + 2 * PF >= ng * PF;
#pragma unroll
      for (int j = 0; j < NTW; ++j) wp[j] = last ? np[j] : wp[j] + 2 * PF * 1024;
      group(ks, p.wa);
      wgroup<0>(wp, p.wa);
      group(ks + PF, p.wb);
      wgroup<PF>(wp, p.wb);
    }
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
      if (tile[j] >= ntl) continue;
      const int n = tile[j] * 16 + 4 * kc;
      const f32x4 bv = bl >= 0 ? *(const f32x4*)(s + bl + 4 * n) : f32x4{0.f, 0.f, 0.f, 0.f};
      epi(lr, n, acc[j], bv);
    }
  }
}

// Forward or input-gradient layer into LDS (see ChainLayer).
// MB: the mask (when there is one) holds a byte per RR rows and column
// instead of elements
template <typename T, int RT, bool FAST, bool MB = false>
__device__ __forceinline__ void run_layer(char* s, const ChainLayer& L, int rv, Pipe& p,
                                          const ChainLayer* next) {
  const int N = L.N;
  const bool relu = L.relu != 0, msk = L.mask.pitch > 0, nopad = L.nopad != 0;
  const LBuf out = L.out, mk = L.mask;
  // Full blocks and widths of whole MFMA depths need no test per element:
  // an add, the max or the mask, the conversion and one store.  The epilogue
  // is vector work that the two product wavefronts of a SIMD mostly do at the
  // same time, so its instructions count beside the MFMAs' cycles (500-1024-512-128
  // at 48 rows per block: k_fwd 121 -> 115 us, k_bwd 83 -> 81; ten 256-wide layers:
  // k_active 70 -> 66, the tick 3 % shorter).  Not at 16 rows per block, where
  // it spilled in k_active and gained nothing elsewhere (20.3 -> 22.0 us).
  const bool whole = RT > 1 && rv == 16 * RT && N % Ch<T>::KS == 0;
  auto epi = [&](int lr, int n, const f32x4 (&a)[RT], const f32x4& b) {
    char* o = lp(s, out, lr, n * (int)sizeof(T));
    const int opitch = 16 * out.pitch;
    if (whole && (MB || !msk)) {
      if (MB && msk) {
        // the 4 columns' bytes of the row's row group in one word, the row's
        // bit of each stretched over the element (the masked value is +0)
        const char* mp = s + mk.off + (lr / Ch<T>::CE) * mk.pitch + n;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const uint32_t w = *(const uint32_t*)(mp + t * (16 / Ch<T>::CE) * mk.pitch) >> (lr % Ch<T>::CE);
          float v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float x0 = a[t][i] + b[i];
            const float x = relu ? fmaxf(x0, 0.f) : x0;
            v[i] = __uint_as_float(__float_as_uint(x) & (uint32_t)((int32_t)(w << (31 - 8 * i)) >> 31));
          }
          st4<T>(o + t * opitch, v);
        }
      } else if (relu) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          float v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = fmaxf(a[t][i] + b[i], 0.f);
          st4<T>(o + t * opitch, v);
        }
      } else {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          float v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = a[t][i] + b[i];
          st4<T>(o + t * opitch, v);
        }
      }
      return;
    }
    // branch-free: every condition is a select (a short-circuit test here
    // compiles to one exec-mask branch per element)
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int r = t * 16 + lr;
      float m[4] = {1.f, 1.f, 1.f, 1.f}, v[4];
      if constexpr (MB) {
        if (msk) {
          const uint32_t w = *(const uint32_t*)(s + mk.off + (r / Ch<T>::CE) * mk.pitch + n);
#pragma unroll
          for (int i = 0; i < 4; ++i) m[i] = (w >> (8 * i + r % Ch<T>::CE)) & 1u ? 1.f : 0.f;
        }
      } else {
        if (msk) ld4<T>(lp(s, mk, r, n * (int)sizeof(T)), m);
      }
      const bool rok = r < rv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x0 = a[t][i] + b[i];
        const float x = relu ? fmaxf(x0, 0.f) : x0;
        const bool keep = rok & (n + i < N) & (m[i] > 0.f);
        v[i] = keep ? x : 0.f;
      }
      // n is a multiple of 4 and a nopad N of 8: the four columns are all
      // below N or all past it
      if (!nopad || n < N) st4<T>(o + t * opitch, v);
    }
  };
  block_mm<T, RT, FAST>(s, L, p, next, epi);
}

// Input gradient of the embedding columns of a bottom input: float32 rows
// of gx (block rows below rv).
template <typename T, int RT, bool FAST>
__device__ __forceinline__ void run_gx(const char* s, const ChainLayer& L, float* gx, int64_t ldgx,
                                       int r0, int rv, Pipe& p) {
  const int N = L.N;
  VFL_GLOBAL float* gxg = glb(gx);
  block_mm<T, RT, FAST>(s, L, p, nullptr, [&](int lr, int n, const f32x4 (&acc)[RT], const f32x4&) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int r = t * 16 + lr;
      const f32x4& a = acc[t];
      if (r >= rv) continue;
      VFL_GLOBAL float* dst = gxg + (int64_t)(r0 + r) * ldgx + n;
      if (n + 4 <= N) {
        *(VFL_GLOBAL f32x4*)dst = a;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < N) dst[i] = a[i];
      }
    }
  });
}

// ------------------------------------------------------------ data movement
// LDS rows -> RC global matrix (block rows at tick rows r0 ..), columns up
// to the next multiple of RR (zero in LDS) included; consecutive lanes store
// consecutive 16-byte chunks (RR rows of one column) of a row group.
// float32: a lane builds a chunk from RR element reads.  bf16: 16 lanes take
// 8 rows x 16 columns with two transposing LDS reads (ds_read_b64_tr_b16:
// lane i of the 16 addresses 4 elements of row i / 4, columns 4 (i mod 4) ..,
// lane j receives column j of the 4 rows), where element reads took eight
// 2-byte reads and their packing per chunk.  The LDS buffers are padded to
// a multiple of the MFMA depth (32 columns), so the 16-column units stay
// inside.  Run by the copy threads.
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// (row, column) of the units u, u + step, ... of a grid of n columns, without
// a division per unit (about 40 instructions for a divisor known at run
// time: more than the copy of a unit)
struct GridWalk {
  int r, c, n, dr, dc;
  __device__ __forceinline__ GridWalk(int u, int n_, int step) : r(u / n_), c(u - r * n_), n(n_), dr(step / n_), dc(step - dr * n_) {}
  __device__ __forceinline__ void next() {
    r += dr;
    c += dc;
    const bool wrap = c >= n;
    r += wrap;
    c -= wrap ? n : 0;
  }
};

// bits 0 and 1: whether the low and the high bf16 of x is positive (sign bit
// clear and not zero; a ReLU output is never NaN)
__device__ __forceinline__ uint32_t positive2(uint32_t x) {
  const uint32_t p = ((x & 0x7fff7fffu) + 0x7fff7fffu) & ~x;   // bits 15 and 31
  return ((p >> 15) & 1u) | ((p >> 30) & 2u);
}

template <typename T, int BR, bool NT>
__device__ __forceinline__ void lds_to_rc_(char* s, const LBuf& b, int cols, const RCMat& m, int r0,
                                           const LBuf& mask, int mcols) {
  constexpr int RR = Ch<T>::CE;
  const int tid = (int)threadIdx.x - kNT, nt = copy_threads();
  const int cw = (cols + RR - 1) / RR * RR;
  const int64_t cp = m.cp;
  VFL_GLOBAL char* g = glb((char*)m.p) + (int64_t)(r0 / RR) * cp * 16;   // the block's first row group
  const int nrg = m.rows > 0 ? min(BR / RR, (m.rows - r0) / RR) : BR / RR;   // row groups inside m
  const bool lds_mask = mask.pitch > 0;
  auto store = [&](int rg, int c, const u32x4& v) {
    VFL_GLOBAL u32x4* dst = (VFL_GLOBAL u32x4*)(g + (uint32_t)((rg * (int)cp + c) * 16));
    if constexpr (NT) __builtin_nontemporal_store(v, dst);
    else *dst = v;
  };
  if constexpr (RR == 8) {
    constexpr int NB = BR > 16 ? 4 : 2;         // units whose LDS reads are in flight together
    const int nc16 = (cw + 15) / 16;
    const int i16 = tid & 15;
    const char* src = s + b.off + (i16 >> 2) * b.pitch + (i16 & 3) * 8;   // the lane's source in unit (0, 0)
    VFL_GLOBAL uint8_t* bits = glb(m.bits) + (int64_t)(r0 / RR) * m.ldb;
    // w: 8 x 16 unit, the same for the 16 lanes
    for (GridWalk w(tid >> 4, nc16, nt >> 4); w.r < nrg;) {
      int rg[NB], c[NB];
      u32x4 v[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        rg[i] = w.r;
        c[i] = 16 * w.c + i16;
        w.next();
        const char* p = src + min(rg[i], nrg - 1) * 8 * b.pitch + (c[i] - i16) * 2;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * b.pitch));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        v[i] = u32x4{l2[0], l2[1], h2[0], h2[1]};
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (rg[i] >= nrg || c[i] >= cw) continue;
        store(rg[i], c[i], v[i]);
        if ((m.bits || lds_mask) && c[i] < mcols) {
          // the chunk's positive rows, one bit each
          const uint32_t byte = positive2(v[i][0]) | positive2(v[i][1]) << 2 | positive2(v[i][2]) << 4 |
                                positive2(v[i][3]) << 6;
          if (m.bits) bits[rg[i] * m.ldb + c[i]] = (uint8_t)byte;
          if (lds_mask) s[mask.off + rg[i] * mask.pitch + c[i]] = (char)byte;
        }
      }
    }
  } else {
    for (GridWalk w(tid, cw, nt); w.r < nrg; w.next()) {
      const int rg = w.r, c = w.c;
      const char* src = s + b.off + rg * RR * b.pitch + c * (int)sizeof(T);
      u32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = *(const uint32_t*)(src + e * b.pitch);
      store(rg, c, v);
      if (lds_mask && c < mcols) {
        uint32_t byte = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) byte |= (uint32_t)(__uint_as_float(v[e]) > 0.f) << e;
        s[mask.off + rg * mask.pitch + c] = (char)byte;
      }
    }
  }
}

// m.p null: nothing; with the streaming hint when m.nt (matrices too large
// for the L2; the two loops are kept apart so that the hint survives).
// mask (its pitch 0: none): the ReLU derivative of the first mcols columns
// (0: cols) as well, in LDS, a byte per RR rows and column.
template <typename T, int BR, bool HINT = false>
__device__ __forceinline__ void lds_to_rc(char* s, const LBuf& b, int cols, const RCMat& m, int r0,
                                          const LBuf& mask = LBuf(), int mcols = 0) {
  if (!m.p) return;
  if (mcols == 0) mcols = cols;
  if constexpr (HINT) {
    if (m.nt) {
      lds_to_rc_<T, BR, true>(s, b, cols, m, r0, mask, mcols);
      return;
    }
  }
  lds_to_rc_<T, BR, false>(s, b, cols, m, r0, mask, mcols);
}

// zero rows r0 .. r0+BR-1 of an RC global matrix (columns below cols)
template <typename T, int BR>
__device__ __forceinline__ void zero_rc(const RCMat& m, int cols, int r0) {
  constexpr int RR = Ch<T>::CE;
  if (!m.p) return;
  const int ncc = (cols + RR - 1) / RR;
  VFL_GLOBAL char* g = glb((char*)m.p);
  const int nrg = m.rows > 0 ? min(BR / RR, (m.rows - r0) / RR) : BR / RR;   // row groups inside m
  for (int u = threadIdx.x; u < nrg * ncc * RR; u += kNT) {
    const int rg = u / (ncc * RR), c = u % (ncc * RR);
    *(VFL_GLOBAL u32x4*)(g + ((int64_t)(r0 / RR + rg) * m.cp + c) * 16) = u32x4{0u, 0u, 0u, 0u};
  }
}

// The ReLU bits of a block's BR rows as they are (a byte per 8 rows and
// column) into b: BR / 8 rows of b.pitch bytes, 16 bytes per lane and load,
// columns up to cols rounded to 16 (within m.ldb), by the copy
// threads.  Row groups past m.rows
// repeat its last (their rows are past the tick's and never kept).
template <int BR>
__device__ __forceinline__ void bits_to_lds(char* s, const LBuf& b, int cols, const RCMat& m, int r0) {
  const int nc = (cols + 15) / 16;
  const int rg_last = m.rows > 0 ? max(m.rows / 8 - 1, 0) : (1 << 30);
  const VFL_GLOBAL uint8_t* bits = glb((const uint8_t*)m.bits);
  for (GridWalk w((int)threadIdx.x - kNT, nc, copy_threads()); w.r < BR / 8; w.next()) {
    const int rg = w.r, c = 16 * w.c;
    const u32x4 v = __builtin_nontemporal_load((const VFL_GLOBAL u32x4*)(bits + (int64_t)min(r0 / 8 + rg, rg_last) * m.ldb + c));
    *(u32x4*)(s + b.off + rg * b.pitch + c) = v;
  }
}

// RC global matrix -> LDS rows (columns below cols; zeros up to the MFMA
// depth), by the copy threads: one 16-byte load per chunk (RR rows of one
// column) and RR element writes, the loads of NB chunks per lane issued
// before their first use (one round trip to HBM per NB chunks).
template <typename T, int BR>
__device__ __forceinline__ void rc_to_lds(char* s, const LBuf& b, int cols, const RCMat& m, int r0) {
  constexpr int RR = Ch<T>::CE, KS = Ch<T>::KS;
  constexpr int NB = 4;
  static_assert(RR == 4, "bf16 masks are bits");
  const int tid = (int)threadIdx.x - kNT, nt = copy_threads();
  const int cw = (cols + KS - 1) / KS * KS;   // columns up to the MFMA depth
  const VFL_GLOBAL char* g = glb((const char*)m.p);
  const int64_t cp = m.cp;
  const int rg_last = m.rows > 0 ? max(m.rows / RR - 1, 0) : (1 << 30);
  const int nu = (BR / RR) * cw;
  for (int u0 = tid; u0 < nu; u0 += NB * nt) {
    u32x4 v[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int u = min(u0 + i * nt, nu - 1);
      const int rg = u / cw, c = min(u - rg * cw, cols - 1);
      v[i] = *(const VFL_GLOBAL u32x4*)(g + ((int64_t)min(r0 / RR + rg, rg_last) * cp + c) * 16);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int u = u0 + i * nt;
      if (u >= nu) continue;
      const int rg = u / cw, c = u - rg * cw;
      const bool ok = c < cols && (m.rows == 0 || r0 + rg * RR < m.rows);
      const u32x4 x = ok ? v[i] : u32x4{0u, 0u, 0u, 0u};
      char* dst = s + b.off + rg * RR * b.pitch + c * (int)sizeof(T);
#pragma unroll
      for (int w = 0; w < 4; ++w) *(uint32_t*)(dst + w * b.pitch) = x[w];
    }
  }
}

// LDS rows -> row-major global rows (16-byte chunks; rows below rv), by the
// copy threads (COPY) or the product threads
template <typename T, int BR, bool COPY>
__device__ __forceinline__ void lds_to_rows(const char* s, const LBuf& b, int cols, void* dst,
                                            int64_t ld, int r0, int rv) {
  const int tid = COPY ? (int)threadIdx.x - kNT : (int)threadIdx.x;
  constexpr int CE = Ch<T>::CE;
  const int nch = (cols + CE - 1) / CE;
  VFL_GLOBAL char* d = glb((char*)dst);
  for (GridWalk w(tid, nch, COPY ? copy_threads() : kNT); w.r < rv; w.next())
    *(VFL_GLOBAL u32x4*)(d + ((int64_t)(r0 + w.r) * ld + w.c * CE) * sizeof(T)) =
        *(const u32x4*)(s + b.off + w.r * b.pitch + w.c * 16);
}

// an embedding id clamped into [0, V)
__device__ __forceinline__ int32_t clamp_id(int32_t id, int32_t V) { return min(max(id, 0), V - 1); }

// Bottom input [embeddings | dense] of the block into LDS (zeros beyond the
// input width up to the MFMA depth and for rows below the group).
template <typename T, int BR>
__device__ __forceinline__ void load_input(char* s, const RowInput& in, const ChainCall& cc,
                                           const Call& k, int r0, int rv) {
  constexpr int CE = Ch<T>::CE, KS = Ch<T>::KS;
  const int ne = in.n_cat * in.E;
  const int din = ne + in.dense_in;
  const int nch = (din + KS - 1) / KS * 4;
  const VFL_GLOBAL T* dense = glb((const T*)cc.dense);
  const VFL_GLOBAL int32_t* ids = glb(cc.ids);
  const VFL_GLOBAL float* tab = glb(in.T);
  if (in.idt) {
    // field-major copy of the block's ids (read contiguously)
    VFL_GLOBAL int32_t* idt = glb(in.idt);
    const VFL_GLOBAL int32_t* src = ids + (k.in_off + r0) * in.n_cat;
    for (int u = threadIdx.x; u < rv * in.n_cat; u += kNT) {
      const int r = u / in.n_cat, f = u - r * in.n_cat;
      int32_t id = src[u];
      if ((uint32_t)id >= (uint32_t)in.V) {
        if (in.bad_ids) atomicAdd(in.bad_ids, 1);
        id = id < 0 ? 0 : in.V - 1;
      }
      idt[(int64_t)f * in.ldi + r0 + r] = id;
    }
  }
  if (ne == 0 && in.dense_vec && BR * nch > kNT) {
    // dense rows only, several chunks per lane: NB chunks per lane in
    // flight before the first LDS write (one round trip to HBM per NB
    // chunks; NB grows with the rows per block, so that narrow blocks keep
    // their register count); chunks past the rows or the width load a valid
    // chunk of the block's first row and store zero.  (With one chunk per
    // lane the loop below issues each lane's only load at once anyway.)
    constexpr int NB = BR / 8 < 8 ? BR / 8 : 8;
    const int nu = BR * nch;
    for (int u0 = threadIdx.x; u0 < nu; u0 += NB * kNT) {
      u32x4 v[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int u = u0 + i * kNT, r = u / nch, c0 = (u % nch) * CE;
        const bool ok = u < nu && r < rv && c0 < din;
        const int64_t row = k.in_off + r0 + (ok ? r : 0);
        v[i] = __builtin_nontemporal_load((const VFL_GLOBAL u32x4*)(dense + row * cc.ld + (ok ? c0 : 0)));
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int u = u0 + i * kNT, r = u / nch, ch = u % nch, c0 = ch * CE;
        if (u >= nu) continue;
        const bool ok = r < rv && c0 < din;
        *(u32x4*)(s + in.buf.off + r * in.buf.pitch + ch * 16) =
            ok ? mask_tail<T>(v[i], din - c0) : u32x4{0u, 0u, 0u, 0u};
      }
    }
    return;
  }
  for (int u = threadIdx.x; u < BR * nch; u += kNT) {
    const int r = u / nch, ch = u % nch, c0 = ch * CE;
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (r < rv && c0 < din) {
      const int64_t row = k.in_off + r0 + r;
      if (c0 >= ne && in.dense_vec && (ne % CE) == 0) {
        v = mask_tail<T>(__builtin_nontemporal_load((const VFL_GLOBAL u32x4*)(dense + row * cc.ld + (c0 - ne))),
                         din - c0);
      } else if (c0 + CE <= ne && (in.E % CE) == 0) {
        const int f = c0 / in.E, o = c0 % in.E;
        const VFL_GLOBAL float* src = tab + ((int64_t)f * in.V + clamp_id(ids[row * in.n_cat + f], in.V)) * in.E + o;
        float x[CE];
#pragma unroll
        for (int q = 0; q < CE / 4; ++q) {
          const f32x4 t = *(const VFL_GLOBAL f32x4*)(src + 4 * q);
          x[4 * q] = t[0]; x[4 * q + 1] = t[1]; x[4 * q + 2] = t[2]; x[4 * q + 3] = t[3];
        }
        if constexpr (sizeof(T) == 4) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(x[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = pack_bf16(x[2 * e], x[2 * e + 1]);
        }
      } else {
        float x[CE];
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          const int c = c0 + e;
          float val = 0.f;
          if (c < ne) {
            const int f = c / in.E;
            val = tab[((int64_t)f * in.V + clamp_id(ids[row * in.n_cat + f], in.V)) * in.E + (c % in.E)];
          } else if (c < din) {
            val = ld1<T>((const T*)(dense + row * cc.ld + (c - ne)));
          }
          x[e] = val;
        }
        if constexpr (sizeof(T) == 4) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(x[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = pack_bf16(x[2 * e], x[2 * e + 1]);
        }
      }
    }
    *(u32x4*)(s + in.buf.off + r * in.buf.pitch + ch * 16) = v;
  }
}

// lane i's value in every lane
__device__ __forceinline__ float lane_value(float x, int i) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), i));
}

// Sums of v[0 .. P-1] over the 64 lanes, P = 2, 4 or 8: lane l returns the
// sum of v[l >> (6 - log2 P)].  A step at lane distance 32, 16 or 8 adds two
// halves of the wavefront and deals the values out between them (the swaps
// exchange a's upper with b's lower lanes); the rest sums in place.  The
// pairs added are those of a butterfly at distances 32, 16, .. 1.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float swap_add32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int P>
__device__ __forceinline__ float rows_reduce(const float (&v)[P], int lane) {
  constexpr int kRor8 = 0x128, kXor2 = 0x4e, kXor1 = 0xb1;   // row_ror:8, quad_perm [2,3,0,1], [1,0,3,2]
  float x;
  if constexpr (P == 2) {
    x = swap_add32(v[0], v[1]);
    x = swap_add16(x, x);
    x += dpp<kRor8>(x);
  } else if constexpr (P == 4) {
    x = swap_add16(swap_add32(v[0], v[2]), swap_add32(v[1], v[3]));
    x += dpp<kRor8>(x);
  } else {
    const float a = swap_add16(swap_add32(v[0], v[4]), swap_add32(v[2], v[6]));
    const float b = swap_add16(swap_add32(v[1], v[5]), swap_add32(v[3], v[7]));
    const bool up = (lane & 8) != 0;
    x = (up ? b : a) + dpp<kRor8>(up ? a : b);
  }
  x += __shfl_xor(x, 4, 64);
  x += dpp<kXor2>(x);
  return x + dpp<kXor1>(x);
}

// Per-row clip + noise of an LDS message of D columns (element V) into
// row-major element-T rows; norm/cfac (nullable) receive ||v|| and the clip
// factor.  16 lanes per row (4 rows per wavefront at a time), each lane on
// the 4-column groups cg, cg + 16, ...; the noise is keyed by the row's
// sample id, two groups' Philox blocks at a time (independent instruction
// streams, so one lane keeps the VALU busy).  Block rows lo .. hi - 1, by
// nwaves wavefronts, this one the wave-th of them.
template <typename V>
__device__ __forceinline__ void msg_ld4(const char* row, int g, int D, float (&x)[4]) {
  ld4<V>(row + 4 * g * (int)sizeof(V), x);
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = 4 * g + e < D ? x[e] : 0.f;   // columns past D may hold anything
}
template <typename T>
__device__ __forceinline__ void msg_st4(VFL_GLOBAL T* o, int g, int D, const float (&v)[4]) {
  if (4 * g + 4 <= D) {
    st4<T>((T*)(o + 4 * g), v);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * g + e < D) st1<T>((T*)(o + 4 * g + e), v[e]);
  }
}
template <typename T, typename V, int BR>
__device__ __forceinline__ void msg_rows(const char* s, const LBuf& src, int D, const MsgOp& m,
                                         uint32_t step, int64_t sample0, void* out, int64_t ldo,
                                         float* norm, float* cfac, int r0, int rv, int wave, int nwaves,
                                         int lo = 0, int hi = BR) {
  const int lane = threadIdx.x & 63;
  const int sub = lane >> 4, cg = lane & 15;
  const int ngrp = (D + 3) >> 2;
  for (int rb = lo; rb < hi; rb += 4 * nwaves) {
    const int r = rb + wave * 4 + sub;
    if (r >= min(rv, hi)) continue;   // uniform within the row's 16 lanes
    const char* row = s + src.off + r * src.pitch;
    float ss = 0.f;
    for (int g = cg; g < ngrp; g += 16) {
      float x[4];
      msg_ld4<V>(row, g, D, x);
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += x[e] * x[e];
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) ss += __shfl_xor(ss, o, 64);
    const float n = sqrtf(ss);
    const float cf = (m.clip && n > m.C) ? m.C / n : 1.f;
    if (cg == 0) {
      if (norm) glb(norm)[r0 + r] = n;
      if (cfac) glb(cfac)[r0 + r] = cf;
    }
    VFL_GLOBAL T* o = glb((T*)out) + (int64_t)(r0 + r) * ldo;
    const uint32_t grow = (uint32_t)(sample0 + r0 + r);
    for (int g = cg; g < ngrp; g += 32) {
      // groups g and g + 16 (the second past the row: computed, never stored)
      float xa[4] = {0.f, 0.f, 0.f, 0.f}, xb[4] = {0.f, 0.f, 0.f, 0.f};
      if (m.noise) {
        gauss4(m.seed, step, grow, (uint32_t)g, m.tag, xa);
        gauss4(m.seed, step, grow, (uint32_t)(g + 16), m.tag, xb);
      }
      float va[4], vb[4];
      msg_ld4<V>(row, g, D, va);
      msg_ld4<V>(row, min(g + 16, ngrp - 1), D, vb);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        va[e] = 4 * g + e < D ? cf * va[e] + m.stdv * xa[e] : 0.f;
        vb[e] = cf * vb[e] + m.stdv * xb[e];
      }
      msg_st4<T>(o, g, D, va);
      if (g + 16 < ngrp) msg_st4<T>(o, g + 16, D, vb);
    }
  }
}

// ------------------------------------------------------------------ kernels
template <typename T, int RT>
__global__ __launch_bounds__(kBT, min_waves(RT, 2)) void k_fwd(const FwdJob* __restrict__ jp, ChainCall cc,
                                             TickRef tr) {
  constexpr int BR = 16 * RT;
  extern __shared__ __attribute__((aligned(16))) char s[];
  const FwdJob& j = *jp;
  const int nL = cst(j).L;
  const Call k = resolve(cc, tr);
  if (blockIdx.x == 0 && threadIdx.x == 0 && j.hdr_out) {
    VFL_GLOBAL int32_t* h = glb(j.hdr_out);
    h[0] = k.hdr[0]; h[1] = k.hdr[1]; h[2] = k.hdr[2];
  }
  const int r0 = blockIdx.x * BR;
  if (r0 >= k.rows) return;
  const int rv = min(BR, k.rows - r0);
  const int din = j.in.n_cat * j.in.E + j.in.dense_in;
  const ChainLayer& last = j.l[nL - 1];
  if (threadIdx.x >= kNT) {
    __syncthreads();
    lds_to_rc<T, BR, true>(s, j.in.buf, din, j.in.rc, r0);
    for (int l = 0; l < nL; ++l) {
      __syncthreads();
      lds_to_rc<T, BR, true>(s, j.l[l].out, j.l[l].N, j.l[l].rc, r0);
    }
    lds_to_rows<T, BR, true>(s, last.out, last.N, j.z, j.ldz, r0, rv);
    return;
  }
  Pipe pp;
  prefetch<T>(&j.l[0], pp);   // overlaps the input rows' loads
  const uint32_t wx = warm_l2(j.warm, jp);
  copy_bias(s, j.bt);
  load_input<T, BR>(s, j.in, cc, k, r0, rv);
  __syncthreads();
  asm volatile("" ::"v"(wx));   // the L2 fetches have landed with the inputs
  for (int l = 0; l < nL; ++l) {
    run_layer<T, RT, RT == 3>(s, j.l[l], rv, pp, l + 1 < nL ? &j.l[l + 1] : nullptr);
    __syncthreads();
  }
  if (j.publish)
    msg_rows<T, T, BR>(s, last.out, last.N, j.m, (uint32_t)k.group, k.row0, j.zhat, j.ldzh, j.norm,
                       j.cfac, r0, rv, (int)(threadIdx.x >> 6), kNW);
}

template <typename T, int RT>
__global__ __launch_bounds__(kBT, min_waves(RT, 1)) void k_active(const ActiveJob* __restrict__ jp, ChainCall cc,
                                                TickRef tr) {
  constexpr int BR = 16 * RT;
  constexpr int CE = Ch<T>::CE, KS = Ch<T>::KS;
  constexpr bool FAST = RT == 3;
  extern __shared__ __attribute__((aligned(16))) char s[];
  const ActiveJob& j = *jp;
  const int LA = cst(j).LA;
  const int H = cst(j).H;
  const int nda = cst(j).nda;
  const int has_gx = cst(j).has_gx;
  const Call k = resolve(cc, tr);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (j.hdr_chk && glb(j.hdr_chk)[0] != k.chk) atomicAdd(j.err, 1);
    if (j.hdr_out) {
      VFL_GLOBAL int32_t* h = glb(j.hdr_out);
      h[0] = k.hdr[0]; h[1] = k.hdr[1]; h[2] = k.hdr[2];
    }
  }
  const int r0 = blockIdx.x * BR;
  if (r0 >= k.rows) {
    // rows past a short group: zero delta rows, so that the weight
    // gradient may read whole row steps
    if (threadIdx.x >= kNT) return;
    zero_rc<T, BR>(j.dh_rc, j.ft[H - 1].N, r0);
    for (int q = 0; q + 1 < H; ++q) zero_rc<T, BR>(j.dt[q].rc, j.dt[q].N, r0);
    zero_rc<T, BR>(j.dc.rc, j.dA, r0);
    for (int q = 0; q < nda; ++q) zero_rc<T, BR>(j.da[q].rc, j.da[q].N, r0);
    return;
  }
  const int rv = min(BR, k.rows - r0);
  const int Hd = j.ft[H - 1].N;
  const int Hd4 = (Hd + 3) / 4 * 4;
  float* yl = (float*)(s + j.red.off);        // the rows' labels
  float* wpart = yl + BR;                     // logit weight gradient [kNW][Hd4]
  float* wl = wpart + kNW * Hd4;              // {loss, dl} [kNW][2]
  const bool gextra = j.gextra != 0;
  // the message with clip or noise: its first rows by the copy wavefronts
  // beside A's input-gradient chain, the others by the product wavefronts
  // after it (64 rows of 128 columns with Philox noise: the copy wavefronts
  // alone took 4.7 us longer than the chain); by all of them together where
  // there is no chain
  const bool msg_all = nda == 0 && !has_gx;
  constexpr int kCopyRows = 16 * (RT > 1 ? RT / 2 : 1);
  auto send_noised = [&](int w0, int nw, int lo, int hi) {
    msg_rows<T, float, BR>(s, j.msg, j.dB, j.m, (uint32_t)k.group, k.row0, j.ring, j.ldring, nullptr, nullptr,
                           r0, rv, wave - w0, nw, lo, hi);
  };
  if (threadIdx.x >= kNT) {
    const int tid = (int)threadIdx.x - kNT, nt = copy_threads();
    // B's embedding into cat[:, dA:dA+dB) with zeros up to the MFMA depth
    // (published before this launch; A's last layer fills cat[:, 0:dA) and
    // leaves these columns alone) and the labels, beside A's input
    {
      const int dA = j.dA, dB = j.dB;
      const int nch = ((dA + dB + KS - 1) / KS * KS - dA) / CE;
      const VFL_GLOBAL T* zb = glb((const T*)j.zb);
      const VFL_GLOBAL float* y = glb(cc.labels) + k.in_off + r0;
      const float py = y[min(tid, rv - 1)];
      for (GridWalk w(tid, nch, nt); w.r < BR; w.next()) {
        const int r = w.r, c = w.c * CE;
        u32x4 v = u32x4{0u, 0u, 0u, 0u};
        if (r < rv && c < dB) v = mask_tail<T>(*(const VFL_GLOBAL u32x4*)(zb + (int64_t)(r0 + r) * j.ldzb + c), dB - c);
        *(u32x4*)(s + j.cat.off + r * j.cat.pitch + (dA + c) * (int)sizeof(T)) = v;
      }
      if (tid < BR) yl[tid] = tid < rv ? py : 0.f;
    }
    // the copy of each stage's output runs beside the next stage
    __syncthreads();
    lds_to_rc<T, BR>(s, j.in.buf, j.in.n_cat * j.in.E + j.in.dense_in, j.in.rc, r0);
    for (int l = 0; l < LA; ++l) {
      __syncthreads();
      // (A's last layer writes cat, copied whole)
      if (l + 1 < LA) lds_to_rc<T, BR>(s, j.fa[l].out, j.fa[l].N, j.fa[l].rc, r0, j.fa[l].mask_out);
      else lds_to_rc<T, BR>(s, j.cat, j.dA + j.dB, j.cat_rc, r0, j.fa[l].mask_out, j.dA);
    }
    for (int q = 0; q < H; ++q) {
      __syncthreads();
      lds_to_rc<T, BR>(s, j.ft[q].out, j.ft[q].N, j.ft[q].rc, r0, j.ft[q].mask_out);
    }
    __syncthreads();
    // the logit stage's sums over the product wavefronts, in order
    VFL_GLOBAL float* part = glb(j.part) + (int64_t)blockIdx.x * (Hd + 2);
    for (int c = tid; c < Hd + 2; c += nt) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < kNW; ++w) t += c < 2 ? wl[2 * w + c] : wpart[w * Hd4 + c - 2];
      part[c] = t;
    }
    lds_to_rc<T, BR>(s, j.dh, Hd, j.dh_rc, r0);
    for (int q = 0; q + 1 < H; ++q) {
      __syncthreads();
      lds_to_rc<T, BR>(s, j.dt[q].out, j.dt[q].N, j.dt[q].rc, r0);
    }
    __syncthreads();
    lds_to_rc<T, BR>(s, j.dc.out, j.dA, j.dc.rc, r0);
    if (gextra && msg_all) send_noised(0, (int)(blockDim.x >> 6), 0, BR);
    else if (gextra) send_noised(kNW, (int)(blockDim.x >> 6) - kNW, 0, kCopyRows);
    else lds_to_rows<T, BR, true>(s, j.msg, j.dB, j.ring, j.ldring, r0, rv);
    for (int q = 0; q < nda; ++q) {
      __syncthreads();
      lds_to_rc<T, BR>(s, j.da[q].out, j.da[q].N, j.da[q].rc, r0);
    }
    return;
  }
  // the logit weights of the lane's columns in the logit stage (columns
  // 256 i + 4 lane .. +4, kept in registers); loads clamped, so all are
  // unconditional
  float lwr[kLogitChunks][4];
  {
    const VFL_GLOBAL float* lw = glb(j.lw);
#pragma unroll
    for (int i = 0; i < kLogitChunks; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 256 * i + 4 * lane + e;
        const float v = lw[min(c, Hd - 1)];
        lwr[i][e] = c < Hd ? v : 0.f;
      }
  }
  const float lbias = glb(j.lb)[0];
  Pipe pp;
  prefetch<T>(&j.fa[0], pp);
  const uint32_t wx = warm_l2(j.warm, jp);
  copy_bias(s, j.bt);

  load_input<T, BR>(s, j.in, cc, k, r0, rv);
  __syncthreads();
  asm volatile("" ::"v"(wx));   // the L2 fetches have landed with the inputs
  for (int l = 0; l < LA; ++l) {
    run_layer<T, RT, FAST>(s, j.fa[l], rv, pp, l + 1 < LA ? &j.fa[l + 1] : &j.ft[0]);
    __syncthreads();
  }
  // top hidden layers
  for (int q = 0; q < H; ++q) {
    run_layer<T, RT, FAST>(s, j.ft[q], rv, pp, q + 1 < H ? &j.ft[q + 1] : (H > 1 ? &j.dt[0] : &j.dc));
    __syncthreads();
  }
  // logit + BCE (Eq. 1), dl = sigmoid(l) - y, or for regression the
  // squared error and dl = 2 (l - y): a wavefront takes BR / 8 rows, lane on
  // the columns 256 i + 4 lane .. +4; the last hidden delta dl * w
  // (ReLU-masked) goes to LDS.  The logit layer's weight gradient
  // sum_r dl_r h[r][c], the loss and dl accumulate per wavefront in
  // registers and are then summed over the wavefronts in order (by the
  // copy wavefronts, beside the next stage).  The loss only reports
  // progress: its exp and log are the hardware's.
  {
    const LBuf Hb = j.ft[H - 1].out, Db = j.dh;
    constexpr int RW = BR / kNW;                // rows per wavefront: 2, 4, 6, 8
    constexpr int P = RW > 4 ? 8 : RW, LP = RW > 4 ? 3 : RW / 2;   // up to a power of two, its log
    const int Hw = (Hd + KS - 1) / KS * KS;     // LDS width of h and dh
    float g[kLogitChunks][4];
#pragma unroll
    for (int i = 0; i < kLogitChunks; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) g[i][e] = 0.f;
    const bool relu_h = j.relu_h != 0;
    auto load_h = [&](int r, float (&h)[kLogitChunks][4]) {
#pragma unroll
      for (int i = 0; i < kLogitChunks; ++i) {
        const int c0 = 256 * i + 4 * lane;
        if (c0 < Hw) ld4<T>(lp(s, Hb, r, c0 * (int)sizeof(T)), h[i]);
        else {
#pragma unroll
          for (int e = 0; e < 4; ++e) h[i][e] = 0.f;
        }
      }
    };
    // the logits of the wavefront's rows: partial dots first, then their
    // sums over the lanes with the rows dealt out on the way (each step
    // halves the rows a lane holds): lane l ends with the logit of row
    // l >> (6 - LP), where a butterfly per row took six shuffles each, and
    // the loss chain below runs once for all rows instead of once per row
    float v[P];
#pragma unroll
    for (int rr = 0; rr < P; ++rr) {
      v[rr] = 0.f;
      if (rr >= RW) continue;
      float h[kLogitChunks][4];
      load_h(wave * RW + rr, h);
#pragma unroll
      for (int i = 0; i < kLogitChunks; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[rr] += h[i][e] * lwr[i][e];
    }
    const float dot = rows_reduce<P>(v, lane);
    // this lane's row: the loss term and dl
    const int lr = lane >> (6 - LP), r = wave * RW + lr;
    const bool ok = lr < RW && r < rv;
    const float l = dot + lbias, yy = yl[min(r, BR - 1)];
    float lt, dl;
    if (cst(j).mse) {
      const float e = l - yy;
      lt = e * e;
      dl = 2.f * e;
    } else {
      const float ex = __expf(-fabsf(l));
      const float inv = __frcp_rn(1.f + ex);
      lt = fmaxf(l, 0.f) - yy * l + __logf(1.f + ex);
      dl = (l >= 0.f ? inv : ex * inv) - yy;
    }
    lt = ok ? lt : 0.f;
    dl = ok ? dl : 0.f;
    float lsum = 0.f, dsum = 0.f;
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      const float dr = lane_value(dl, rr << (6 - LP));
      lsum += lane_value(lt, rr << (6 - LP));
      dsum += dr;
      float h[kLogitChunks][4];
      load_h(wave * RW + rr, h);
#pragma unroll
      for (int i = 0; i < kLogitChunks; ++i) {
        const int c0 = 256 * i + 4 * lane;
        float d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          d[e] = dr * lwr[i][e];
          if (relu_h && !(h[i][e] > 0.f)) d[e] = 0.f;
          g[i][e] += dr * h[i][e];
        }
        if (c0 < Hw) st4<T>(lp(s, Db, wave * RW + rr, c0 * (int)sizeof(T)), d);
      }
    }
#pragma unroll
    for (int i = 0; i < kLogitChunks; ++i) {
      const int c0 = 256 * i + 4 * lane;
      if (c0 < Hd4) *(f32x4*)(wpart + wave * Hd4 + c0) = f32x4{g[i][0], g[i][1], g[i][2], g[i][3]};
    }
    if (lane == 0) {
      wl[2 * wave] = lsum;
      wl[2 * wave + 1] = dsum;
    }
    __syncthreads();
  }
  // top input-gradient chain
  for (int q = 0; q + 1 < H; ++q) {
    run_layer<T, RT, FAST, true>(s, j.dt[q], rv, pp, q + 2 < H ? &j.dt[q + 1] : &j.dc);
    __syncthreads();
  }
  // concat product: A's cut delta and the gradient message for B
  {
    const int dA = j.dA, dAB = j.dA + j.dB;
    const int dApad = (dA + KS - 1) / KS * KS;
    const LBuf ob = j.dc.out, mk = j.dc.mask, msg = j.msg;
    const bool maskA = mk.pitch > 0;
    const int msg_end = dA + (j.dB + CE - 1) / CE * CE;   // the message's columns in whole chunks
    block_mm<T, RT, FAST>(s, j.dc, pp, nda > 0 ? &j.da[0] : (has_gx ? &j.gx : nullptr),
                    [&](int lr, int n, const f32x4 (&acc)[RT], const f32x4&) {
#pragma unroll
     for (int t = 0; t < RT; ++t) {
      const int r = t * 16 + lr;
      const f32x4& a = acc[t];
      const bool ok = r < rv;
      if (n < dA) {   // dA is a multiple of 8: all four columns are A's
        uint32_t w = ~0u;
        float v[4];
        if (maskA) w = *(const uint32_t*)(s + mk.off + (r / CE) * mk.pitch + n);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (ok && ((w >> (8 * i + r % CE)) & 1u)) ? a[i] : 0.f;
        st4<T>(lp(s, ob, r, n * (int)sizeof(T)), v);
        continue;
      }
      // the message to LDS (float32 when clip or noise follow), where the
      // copy wavefronts take it from
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = ok && n + i < dAB ? a[i] : 0.f;
      if (n < dApad) {
#pragma unroll
        for (int i = 0; i < 4; ++i) st1<T>((T*)lp(s, ob, r, 0) + n + i, 0.f);
      }
      if (n < msg_end) {
        if (gextra) st4<float>(lp(s, msg, r, (n - dA) * 4), v);
        else st4<T>(lp(s, msg, r, (n - dA) * (int)sizeof(T)), v);
      }
     }
    });
    __syncthreads();
    if (gextra && msg_all) send_noised(0, (int)(blockDim.x >> 6), 0, BR);
  }
  // A's input-gradient chain
  for (int q = 0; q < nda; ++q) {
    run_layer<T, RT, FAST, true>(s, j.da[q], rv, pp, q + 1 < nda ? &j.da[q + 1] : (has_gx ? &j.gx : nullptr));
    __syncthreads();
  }
  if (has_gx) run_gx<T, RT, FAST>(s, j.gx, j.gxp, j.ldgx, r0, rv, pp);
  if (gextra && !msg_all && kCopyRows < BR) send_noised(0, kNW, kCopyRows, BR);
}

template <typename T, int RT>
__global__ __launch_bounds__(kBT, min_waves(RT, 2)) void k_bwd(const BwdJob* __restrict__ jp, ChainCall cc,
                                             TickRef tr) {
  constexpr int BR = 16 * RT;
  constexpr int KS = Ch<T>::KS;
  extern __shared__ __attribute__((aligned(16))) char s[];
  const BwdJob& j = *jp;
  const int nd = cst(j).nd;
  const int has_gx = cst(j).has_gx;
  const Call k = resolve(cc, tr);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blockIdx.x == 0 && threadIdx.x == 0 && j.hdr_chk && glb(j.hdr_chk)[0] != k.chk) atomicAdd(j.err, 1);
  const int r0 = blockIdx.x * BR;
  if (r0 >= k.rows) {
    if (threadIdx.x >= kNT) return;
    zero_rc<T, BR>(j.d_rc, j.D, r0);
    for (int q = 0; q < nd; ++q) zero_rc<T, BR>(j.dx[q].rc, j.dx[q].N, r0);
    return;
  }
  const int rv = min(BR, k.rows - r0);
  if (threadIdx.x >= kNT) {
    // the ReLU masks of every layer of the chain, each in an LDS buffer of
    // its own (bf16: the ReLU bits of this group's forward as bytes; float32:
    // its stashed activations), beside the cut layer
    for (int q = 0; q < j.nmask; ++q) {
      if constexpr (sizeof(T) == 2) bits_to_lds<BR>(s, j.ml[q].b, j.ml[q].cols, j.ml[q].m, r0);
      else rc_to_lds<T, BR>(s, j.ml[q].b, j.ml[q].cols, j.ml[q].m, r0);
    }
    __syncthreads();
    lds_to_rc<T, BR, true>(s, j.d, j.D, j.d_rc, r0);
    for (int q = 0; q < nd; ++q) {
      __syncthreads();
      lds_to_rc<T, BR, true>(s, j.dx[q].out, j.dx[q].N, j.dx[q].rc, r0);
    }
    return;
  }
  Pipe pp;
  if (nd > 0 || has_gx) prefetch<T>(nd > 0 ? &j.dx[0] : &j.gx, pp);
  const uint32_t wx = warm_l2(j.warm, jp);
  // cut-layer backward: through the clip when the row was clipped
  // (d(c v)/dv = c (I - u u^T) with u = v / ||v||), then the ReLU of B's
  // last layer; 16 lanes per row, 4 rows per wavefront at a time
  {
    const int D = j.D;
    const int hq = (D + KS - 1) / KS * KS / 4;
    const int sub = lane >> 4, cg = lane & 15;
    for (int rb = 0; rb < BR; rb += 4 * kNW) {
      const int r = rb + wave * 4 + sub;
      if (r >= BR) continue;   // uniform within the row's 16 lanes
      const bool ok = r < rv;
      const int64_t row = r0 + r;
      const VFL_GLOBAL T* G = glb((const T*)j.g) + row * j.ldg;
      const VFL_GLOBAL T* Z = glb((const T*)j.z) + row * j.ldz;
      const bool clipped = ok && j.clip && glb(j.norm)[row] > j.C;
      float dot = 0.f, inv = 0.f, cf = 1.f;
      if (clipped) {
        inv = 1.f / glb(j.norm)[row];
        cf = glb(j.cfac)[row];
        for (int q = cg; 4 * q < D; q += 16)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (4 * q + e < D) dot += ld1<T>((const T*)(Z + 4 * q + e)) * inv * ld1<T>((const T*)(G + 4 * q + e));
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) dot += __shfl_xor(dot, o, 64);
      }
      for (int q = cg; q < hq; q += 16) {
        float gv[4] = {0.f, 0.f, 0.f, 0.f}, zv[4] = {0.f, 0.f, 0.f, 0.f}, v[4];
        if (ok && 4 * q + 4 <= D) {
          ld4<T>((const T*)(G + 4 * q), gv);
          ld4<T>((const T*)(Z + 4 * q), zv);
        } else if (ok) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (4 * q + e < D) { gv[e] = ld1<T>((const T*)(G + 4 * q + e)); zv[e] = ld1<T>((const T*)(Z + 4 * q + e)); }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float g = gv[e];
          if (clipped) g = cf * (g - zv[e] * inv * dot);
          if (j.relu && !(zv[e] > 0.f)) g = 0.f;
          v[e] = (ok && 4 * q + e < D) ? g : 0.f;
        }
        st4<T>(lp(s, j.d, r, 4 * q * (int)sizeof(T)), v);
      }
    }
  }
  __syncthreads();
  asm volatile("" ::"v"(wx));   // the L2 fetches have landed with the inputs
  for (int q = 0; q < nd; ++q) {
    const ChainLayer& L = j.dx[q];
    run_layer<T, RT, RT == 3, sizeof(T) == 2>(s, L, rv, pp, q + 1 < nd ? &j.dx[q + 1] : (has_gx ? &j.gx : nullptr));
    __syncthreads();
  }
  if (has_gx) run_gx<T, RT, RT == 3>(s, j.gx, j.gxp, j.ldgx, r0, rv, pp);
  if (j.drm) {
    // the last delta of the chain, row-major, for the layer product below it
    const LBuf last = nd > 0 ? j.dx[nd - 1].out : j.d;
    const int w = nd > 0 ? j.dx[nd - 1].N : j.D;
    lds_to_rows<T, BR, false>(s, last, w, j.drm, j.lddrm, r0, rv);
  }
}

template <typename K>
hipError_t raise_lds(K kernel) {
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
}

}  // namespace


#define VFL_CHAIN_RT(K, T, rt, ...)                                                         \
  do {                                                                                     \
    if (rt == 1) hipLaunchKernelGGL((K<T, 1>), __VA_ARGS__);                               \
    else if (rt == 2) hipLaunchKernelGGL((K<T, 2>), __VA_ARGS__);                          \
    else if (rt == 3) hipLaunchKernelGGL((K<T, 3>), __VA_ARGS__);                          \
    else if (rt == 4) hipLaunchKernelGGL((K<T, 4>), __VA_ARGS__);                          \
    else return hipErrorInvalidValue;                                                      \
  } while (0)
#define VFL_CHAIN(K, e, rt, ...)                                                            \
  do {                                                                                     \
    if (lds > kLdsMax || blocks < 1) return hipErrorInvalidValue;                          \
    const dim3 thr(kBT);                                                                   \
    if (e == BF16) VFL_CHAIN_RT(K, uint16_t, rt, dim3(blocks), thr, __VA_ARGS__);          \
    else VFL_CHAIN_RT(K, float, rt, dim3(blocks), thr, __VA_ARGS__);                       \
  } while (0)

hipError_t launch_fwd(Elt e, int rt, const FwdJob* job, int lds, int blocks, const ChainCall& c,
                      TickRef tr, hipStream_t st) {
  VFL_CHAIN(k_fwd, e, rt, lds, st, job, c, tr);
  return hipGetLastError();
}

hipError_t launch_active(Elt e, int rt, const ActiveJob* job, int lds, int blocks,
                         const ChainCall& c, TickRef tr, hipStream_t st) {
  VFL_CHAIN(k_active, e, rt, lds, st, job, c, tr);
  return hipGetLastError();
}

hipError_t launch_bwd(Elt e, int rt, const BwdJob* job, int lds, int blocks, const ChainCall& c,
                      TickRef tr, hipStream_t st) {
  VFL_CHAIN(k_bwd, e, rt, lds, st, job, c, tr);
  return hipGetLastError();
}

namespace {
template <typename T, int RT>
hipError_t raise_lds_rt() {
  for (hipError_t e : {raise_lds(k_fwd<T, RT>), raise_lds(k_active<T, RT>), raise_lds(k_bwd<T, RT>)})
    if (e != hipSuccess) return e;
  return hipSuccess;
}
template <typename T>
hipError_t raise_lds_all() {
  for (hipError_t e : {raise_lds_rt<T, 1>(), raise_lds_rt<T, 2>(), raise_lds_rt<T, 3>(), raise_lds_rt<T, 4>()})
    if (e != hipSuccess) return e;
  return hipSuccess;
}
}  // namespace

hipError_t chain_init() {
  for (hipError_t e : {raise_lds_all<uint16_t>(), raise_lds_all<float>(), dwt_init(), lin_init()})
    if (e != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace vfl
