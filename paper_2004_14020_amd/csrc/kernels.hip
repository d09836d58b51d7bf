// gfx950 kernels of the aggregation path.  Everything here is bandwidth work: 128-bit
// coalesced loads and stores, no matrix cores.
//
//  k_walk, k_tree_walk, k_ring_reduce, k_ring_reduce_tree_any
//                  ring reduce-scatter arithmetic, 1/W scaling and all-gather (paper
//                  sections 2 and 4.4: partial sums travel round the ring and are added to
//                  at each worker; the owner's result is then copied to every worker).
//                  A workgroup handles one tile: long tiles one replica after the other (chains:
//                  k_walk, trees: k_tree_walk), small ones with all replicas at once.
//  k_slices, k_slice, k_tree_slices, k_tree_slice
//                  the same arithmetic for small jobs, whose work is cut into 1 KiB slices: a wavefront
//                  takes several of them, of whatever tensors and segments, from a table of addresses.
//  k_slice_table   writes that table, once per bind.
//  k_copy          pack / unpack of batched parameters (section 4.2) through an offset table,
//                  one workgroup per run of at most 16 KiB.
#include "kernels.hpp"

#include <type_traits>
#include <utility>

namespace caramel {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// Pointers built from table entries are declared as global-memory pointers so that loads and
// stores use the global (scalar base + lane offset) form rather than the generic one.
#define CARAMEL_GLOBAL __attribute__((address_space(1)))
typedef CARAMEL_GLOBAL u32x4* gvec_ptr;
typedef CARAMEL_GLOBAL float* gf32_ptr;
typedef CARAMEL_GLOBAL uint16_t* gu16_ptr;
typedef CARAMEL_GLOBAL uint32_t* gu32_ptr;

constexpr int kCopyBlock = 1024;  // pack / unpack workgroup
constexpr int kMaxBlock = 1024;  // ring-reduce workgroups are 256, 512 or 1024 lanes

// scalar base + 32-bit lane byte offset
__device__ __forceinline__ gvec_ptr at(gvec_ptr base, uint32_t byte_off) {
  return reinterpret_cast<gvec_ptr>(reinterpret_cast<CARAMEL_GLOBAL char*>(base) + byte_off);
}

// The buffer accesses take the cache policy as an operand: `nt` and `sc1` bits.
constexpr int kNt = 2, kSc1 = 16;
template <int P>
constexpr int kLoadBits = P == kPlain ? 0 : kNt;
template <int P>
constexpr int kStoreBits = P == kPlain ? 0 : (P == kThrough ? kSc1 | kNt : kNt);
constexpr int kRawBuffer = 0x00027000;  // word 3 of a buffer resource: untyped data

template <int P>
__device__ __forceinline__ u32x4 ld(gvec_ptr p) {
  if constexpr (P != kPlain) return __builtin_nontemporal_load(p);
  else return *p;
}
template <int P>
__device__ __forceinline__ void st(gvec_ptr p, u32x4 v) {
  static_assert(P != kThrough, "needs the form with a base and an offset");
  if constexpr (P == kStream) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <int P>
__device__ __forceinline__ void st(gvec_ptr base, uint32_t byte_off, u32x4 v) {
  if constexpr (P == kThrough) {
    // C++ has no way to ask for this pair on a 128-bit store; the buffer form takes the policy as an
    // operand.  The resource is the bare base (untyped, no bound of its own).
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, kRawBuffer);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, int(byte_off), 0, kStoreBits<P>);
  } else {
    st<P>(at(base, byte_off), v);
  }
}

__device__ __forceinline__ f32x4 bits_to_f32(u32x4 v) { return __builtin_bit_cast(f32x4, v); }
__device__ __forceinline__ u32x4 f32_to_bits(f32x4 v) { return __builtin_bit_cast(u32x4, v); }

// fp32 -> bf16, round to nearest, ties to even; NaN stays a (quiet) NaN.  Two values to a conversion
// instruction (it equals the integer arithmetic  (b + 0x7FFF + (b >> 16 & 1)) >> 16,  NaN: b >> 16 | 0x40;
// tests/test_gpu_rounding.py), where that arithmetic takes six instructions a value.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ uint32_t bf16_rne(float f) { return bf16_pair(f, f) & 0xFFFFu; }

// Running ring sum of one 16-byte vector.  F32: four lanes.  BF16: eight values, kept as the
// even-indexed (low halves) and odd-indexed (high halves) quartets, widened exactly.
template <bool BF16>
struct Chain {
  f32x4 a, b;
  __device__ __forceinline__ void start(u32x4 x) {
    if constexpr (BF16) {
      a = bits_to_f32(x << 16);
      b = bits_to_f32(x & 0xFFFF0000u);
    } else {
      a = bits_to_f32(x);
    }
  }
  __device__ __forceinline__ void add(u32x4 x) {
    if constexpr (BF16) {
      a = a + bits_to_f32(x << 16);
      b = b + bits_to_f32(x & 0xFFFF0000u);
    } else {
      a = a + bits_to_f32(x);
    }
  }
  // this partial sum + another one
  __device__ __forceinline__ void merge(const Chain& o) {
    a = a + o.a;
    if constexpr (BF16) b = b + o.b;
  }
  // the sum of no values: -0.0, which leaves every first value as it is
  __device__ __forceinline__ void zero() {
    a = f32x4{-0.0f, -0.0f, -0.0f, -0.0f};
    if constexpr (BF16) b = a;
  }
  // add() in the lanes where `c` holds; the others add -0.0, which changes nothing
  __device__ __forceinline__ void add_if(bool c, u32x4 x) {
    constexpr uint32_t kNothing = BF16 ? 0x80008000u : 0x80000000u;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = c ? x[i] : kNothing;
    add(x);
  }
  // the sum is formed here: left to itself, the compiler moves the additions of an unrolled walk behind
  // its last load, and every value it has loaded stays live until then
  __device__ __forceinline__ void pin() {
    asm volatile("" : "+v"(a));
    if constexpr (BF16) asm volatile("" : "+v"(b));
  }
  __device__ __forceinline__ u32x4 finish(float inv_w) {
    if constexpr (BF16) {
      const f32x4 ya = a * inv_w, yb = b * inv_w;
      u32x4 r;
      r.x = bf16_pair(ya.x, yb.x);
      r.y = bf16_pair(ya.y, yb.y);
      r.z = bf16_pair(ya.z, yb.z);
      r.w = bf16_pair(ya.w, yb.w);
      return r;
    } else {
      return f32_to_bits(a * inv_w);
    }
  }
};

// Sum of the W vectors x[0..W-1] in the order of the pattern, scaled and converted back.
// Chain: ((x0 + x1) + x2) + ...   Tree: neighbours first, then pairs of pairs, ...
template <int W, bool BF16, bool TREE>
__device__ __forceinline__ u32x4 combine(const u32x4 (&x)[W], float inv_w) {
  if constexpr (!TREE) {
    Chain<BF16> c;
    c.start(x[0]);
#pragma unroll
    for (int k = 1; k < W; ++k) c.add(x[k]);
    return c.finish(inv_w);
  } else {
    Chain<BF16> part[W];
#pragma unroll
    for (int k = 0; k < W; ++k) part[k].start(x[k]);
#pragma unroll
    for (int s = 1; s < W; s *= 2)
#pragma unroll
      for (int i = 0; i + s < W; i += 2 * s) {
        part[i].a = part[i].a + part[i + s].a;
        if constexpr (BF16) part[i].b = part[i].b + part[i + s].b;
      }
    return part[0].finish(inv_w);
  }
}

// Same for one scalar element per worker.
template <int W, bool TREE>
__device__ __forceinline__ float combine_scalar(float (&v)[W], float inv_w) {
  if constexpr (!TREE) {
    float acc = v[0];
#pragma unroll
    for (int k = 1; k < W; ++k) acc = acc + v[k];
    return acc * inv_w;
  } else {
#pragma unroll
    for (int s = 1; s < W; s *= 2)
#pragma unroll
      for (int i = 0; i + s < W; i += 2 * s) v[i] = v[i] + v[i + s];
    return v[0] * inv_w;
  }
}

__device__ __forceinline__ float widen(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// ------------------------------------------------------------------------------------------
// W known at compile time: all W loads of a vector (times U vectors) are issued before the
// first add, so each lane keeps W*U 128-bit requests in flight.
template <int W, int U, bool BF16, int P, bool TREE>
__global__ void __launch_bounds__(kMaxBlock)
k_ring_reduce(const ReduceTile* __restrict__ tiles, const uint64_t* __restrict__ rows, uint32_t begin,
              uint32_t count, float inv_w) {
  constexpr uint32_t VE = BF16 ? 8 : 4;
  for (uint32_t ti = blockIdx.x; ti < count; ti += gridDim.x) {
    const ReduceTile tl = tiles[begin + ti];
    gvec_ptr p[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
      uint32_t w = tl.first + k;
      if (w >= uint32_t(W)) w -= W;
      p[k] = reinterpret_cast<gvec_ptr>(rows[size_t(tl.row) * W + w]) + tl.vec_off;
    }
    const uint32_t nvec = tl.n_elems / VE;
    const uint32_t B = blockDim.x;
    uint32_t v = threadIdx.x;
    // lane offsets are 32-bit byte offsets from the scalar bases (a tile spans < 2^24 bytes)
    for (; v + (U - 1) * B < nvec; v += U * B) {
      u32x4 x[U][W];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < W; ++k) x[u][k] = ld<P>(at(p[k], (v + u * B) * 16u));
      __builtin_amdgcn_sched_barrier(0);  // keep all loads ahead of the arithmetic
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const u32x4 y = combine<W, BF16, TREE>(x[u], inv_w);
#pragma unroll
        for (int k = 0; k < W; ++k) st<P>(p[k], (v + u * B) * 16u, y);
      }
    }
    for (; v < nvec; v += B) {
      u32x4 x[W];
#pragma unroll
      for (int k = 0; k < W; ++k) x[k] = ld<P>(at(p[k], v * 16u));
      __builtin_amdgcn_sched_barrier(0);
      const u32x4 y = combine<W, BF16, TREE>(x, inv_w);
#pragma unroll
      for (int k = 0; k < W; ++k) st<P>(p[k], v * 16u, y);
    }
    // a run that ends a tensor may stop inside a vector: finish it element by element
    const uint32_t rem = tl.n_elems - nvec * VE;
    if (threadIdx.x < rem) {
      const uint32_t e = nvec * VE + threadIdx.x;
      float v[W];
      if constexpr (BF16) {
#pragma unroll
        for (int k = 0; k < W; ++k) v[k] = widen(reinterpret_cast<gu16_ptr>(p[k])[e]);
        const uint16_t y = uint16_t(bf16_rne(combine_scalar<W, TREE>(v, inv_w)));
#pragma unroll
        for (int k = 0; k < W; ++k) reinterpret_cast<gu16_ptr>(p[k])[e] = y;
      } else {
#pragma unroll
        for (int k = 0; k < W; ++k) v[k] = reinterpret_cast<gf32_ptr>(p[k])[e];
        const float y = combine_scalar<W, TREE>(v, inv_w);
#pragma unroll
        for (int k = 0; k < W; ++k) reinterpret_cast<gf32_ptr>(p[k])[e] = y;
      }
    }
  }
}

// Chain orders, one replica after the other (long tiles of any W up to 64, and the small tiles of the
// world sizes without a kernel of their own).
//
// Bound: HBM.  A 1024-lane workgroup asks for N * 16 KiB contiguous bytes of one replica, then of the
// next, ...: it issues the next worker's N loads at once, then waits for the current worker's and adds
// them.  The memory system serves such bursts best: an in-place update of 8 x 512 MiB (16 x 94 MiB)
// reaches 82.5 (79.0) % of 8 TB/s with N = 8 and 79.1 (77.3) with N = 4; with each load re-issued as
// soon as its own values were added, which keeps as many bytes in flight, 76.2 (74.0).
//
// The tile is a buffer resource of its own size in every replica: a lane beyond the end of a ragged
// last row reads zeros that nothing uses and its stores are dropped, without a branch, and the loads
// take no address registers: two sets of eight vectors and eight fp32 sums fit 128 VGPRs (four vectors
// with bf16, whose sums take twice the room).  Unrolled over the workers up to 8; over 16 the bases no
// longer fit beside the sums (8 VGPRs and 28 SGPRs spilled), and the rolled loop is no slower
// (ResNet-v2-152 1263 -> 1258 us, Inception-v3 512 -> 510, bf16 16 x 33 MiB 203.6 -> 202.5).
constexpr uint32_t kNowhere = 0x40000000u;  // an offset beyond every tile

// The segment boundaries inside a tile, in bytes from its start.
struct Splits {
  uint32_t n;
  uint32_t at[kMaxSplits];
  __device__ __forceinline__ explicit Splits(const ReduceTile& t, uint32_t elem_bytes) : n(0) {
#pragma unroll
    for (uint32_t i = 0; i < kMaxSplits; ++i) {
      const uint32_t b = i == 0 ? t.split : t.more[i == 0 ? 0 : i - 1];
      at[i] = b ? b * elem_bytes : ~0u;
      n += b ? 1u : 0u;
    }
  }
  // how many of them lie at or before `off`
  __device__ __forceinline__ uint32_t before(uint32_t off) const {
    uint32_t s = 0;
#pragma unroll
    for (uint32_t i = 0; i < kMaxSplits; ++i) s += off >= at[i] ? 1u : 0u;
    return s;
  }
};

// One tile's chain.  CW: the number of workers, 0 if known at run time only (the loop over them is
// rolled then).
// SPLIT (a tile across S segment boundaries, S < W; CW == 0): the workers are visited in the
// tile's order and then the first S once more, W + S steps; a lane behind s of the boundaries, whose
// sums start s workers later, adds the values of steps s .. s+W-1.  A lane asks for no data in the
// steps it sits out, so nothing is fetched twice and the whole workgroup still reads one replica at a
// time.
template <int CW, bool BF16, int P, bool SPLIT>
struct Walk {
  static_assert(!SPLIT || CW == 0, "the unrolled loop has no room for the conditions");
  const uint64_t* __restrict__ row;
  uint64_t mine;       // CW == 0: the tile's address in replica `lane` (W <= 64: every wavefront holds all)
  uint64_t start;      // bytes from a row's base to the tile
  uint32_t workers, first, bytes;
  const Splits& splits;
  float inv_w;

  __device__ __forceinline__ uint32_t W() const { return CW ? uint32_t(CW) : workers; }
  __device__ __forceinline__ uint32_t steps() const { return W() + (SPLIT ? splits.n : 0u); }
  __device__ __forceinline__ uint32_t worker(uint32_t k) const {  // k < 2 W
    uint32_t w = first + k;
    if (SPLIT && w >= 2 * W()) w -= W();
    return w >= W() ? w - W() : w;
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t res(uint32_t w) const {  // the tile in replica w
    uint64_t base;
    if constexpr (CW == 0) {
      // from the lane that keeps it: no scalar load to wait for at every step
      base = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(mine >> 32), int(w)))) << 32 |
             uint32_t(__builtin_amdgcn_readlane(int(mine), int(w)));
    } else {
      base = row[w] + start;
    }
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base), 0, int(bytes), kRawBuffer);
  }

  // One pass over N vectors of this lane: `off` + u * `stride`, in bytes from the tile's start.
  template <int N>
  __device__ __forceinline__ void rows(uint32_t off, uint32_t stride) const {
    const uint32_t n_steps = steps();
    uint32_t lateness = 0;  // boundaries before each of the N vectors, four bits each
    if constexpr (SPLIT) {
#pragma unroll
      for (int u = 0; u < N; ++u) lateness |= splits.before(off + u * stride) << (4 * u);
    }
    auto wanted = [&](uint32_t k, int u) -> bool {  // step k adds to vector u
      return !SPLIT || k - ((lateness >> (4 * u)) & 15u) < W();  // (unsigned: false for k < lateness)
    };
    Chain<BF16> acc[N];
    u32x4 buf[2][N];
#pragma unroll
    for (int u = 0; u < N; ++u) acc[u].zero();
    auto load = [&](uint32_t k, int j) {
      const __amdgpu_buffer_rsrc_t r = res(worker(k));
      if constexpr (SPLIT) asm volatile("" : "+v"(lateness));  // (shifted anew: no registers for the parts)
#pragma unroll
      for (int u = 0; u < N; ++u)
        buf[j][u] = __builtin_amdgcn_raw_buffer_load_b128(r, int(wanted(k, u) ? off + u * stride : kNowhere), 0, kLoadBits<P>);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto add = [&](uint32_t k, int j) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if constexpr (SPLIT) acc[u].add_if(wanted(k, u), buf[j][u]);
        else acc[u].add(buf[j][u]);
        acc[u].pin();
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    load(0, 0);
    if constexpr (CW != 0) {
      #pragma unroll
      for (int k = 0; k < CW; ++k) {
        if (k + 1 < CW) load(k + 1, (k + 1) % 2);
        add(k, k % 2);
      }
    } else {
      uint32_t k = 0;
#pragma unroll 1
      for (; k + 2 < n_steps; k += 2) {
        load(k + 1, 1);
        add(k, 0);
        load(k + 2, 0);
        add(k + 1, 1);
      }
      if (k + 1 < n_steps) load(k + 1, 1);
      add(k, 0);
      if (k + 1 < n_steps) add(k + 1, 1);
    }
    u32x4 y[N];
#pragma unroll
    for (int u = 0; u < N; ++u) y[u] = acc[u].finish(inv_w);
#pragma unroll(CW ? CW : 4)
    for (uint32_t k = 0; k < W(); ++k) {
      const __amdgpu_buffer_rsrc_t r = res(worker(k));
#pragma unroll
      for (int u = 0; u < N; ++u) __builtin_amdgcn_raw_buffer_store_b128(y[u], r, int(off + u * stride), 0, kStoreBits<P>);
    }
  }

  // One vector per lane: nothing to walk, the workers' values are fetched up to sixteen at a time.
  __device__ __forceinline__ void column(uint32_t off) const {
    constexpr int kMost = CW ? CW : 16;
    const uint32_t n_steps = steps(), late = SPLIT ? splits.before(off) : 0;
    Chain<BF16> acc;
    acc.zero();
    for (uint32_t k0 = 0; k0 < n_steps; k0 += kMost) {
      u32x4 x[kMost];
#pragma unroll
      for (int i = 0; i < kMost; ++i)
        if (CW || i == 0 || k0 + i < n_steps) {
          const bool wanted = !SPLIT || k0 + i - late < W();
          x[i] = __builtin_amdgcn_raw_buffer_load_b128(res(worker(k0 + i)), int(wanted ? off : kNowhere), 0, kLoadBits<P>);
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kMost; ++i)
        if (CW || i == 0 || k0 + i < n_steps) {
          if constexpr (SPLIT) acc.add_if(k0 + i - late < W(), x[i]);
          else acc.add(x[i]);
        }
    }
    const u32x4 y = acc.finish(inv_w);
#pragma unroll(CW ? CW : 4)
    for (uint32_t k = 0; k < W(); ++k)
      __builtin_amdgcn_raw_buffer_store_b128(y, res(worker(k)), int(off), 0, kStoreBits<P>);
  }
};

// MAXN: most vectors per lane and pass (long tiles: 8 with fp32, 4 with bf16; small ones: 1); `cap`
// lowers it.
// A walk over long tiles asks for at most four wavefronts per SIMD, one 1024-lane workgroup per compute
// unit, which most of them need anyway (65 to 128 VGPRs).  With two workers and bf16 60 would do, and two
// workgroups then read and write in step: 2 x 33 MiB 27.5 us, 25.8 with one, 2 x 260 MiB 174.3 / 171.0.
// It also leaves the compiler room between the loads (8 workers bf16, 260 MiB: 714.6 / 703.2).
template <int CW, bool BF16, int P, int MAXN>
__global__ void __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(4, MAXN > 1 ? 4 : 8)))
k_walk(const ReduceTile* __restrict__ tiles, const uint64_t* __restrict__ rows, uint32_t begin, uint32_t count,
       uint32_t workers, uint32_t cap, float inv_w) {
  constexpr uint32_t VE = BF16 ? 8 : 4;
  constexpr bool kSplits = CW == 0 || CW == 3;  // (1, 2, 4 and 8 workers: no tile holds a boundary)
  const uint32_t W = CW ? uint32_t(CW) : workers;
  for (uint32_t ti = blockIdx.x; ti < count; ti += gridDim.x) {
    const ReduceTile tl = tiles[begin + ti];
    const uint64_t* row = rows + size_t(tl.row) * W;
    const uint32_t nvec = tl.n_elems / VE;
    const uint32_t B = blockDim.x;
    const uint64_t start = uint64_t(tl.vec_off) * 16;
    const Splits splits(tl, 16 / VE);
    const uint32_t lane = threadIdx.x % 64;
    const uint64_t mine = CW == 0 || (kSplits && tl.split) ? row[lane < W ? lane : W - 1] + start : 0;
    const uint32_t total_rows = (nvec + B - 1) / B;
    for (uint32_t done = 0; done < total_rows;) {
      const uint32_t left = total_rows - done;
      // (three workers: the few tiles with a boundary take two passes; eight vectors of that walk beside the
      // unrolled one spill)
      const uint32_t most = CW == 3 && MAXN > 4 && tl.split && cap > 4 ? 4 : cap;
      const uint32_t n = left < most ? left : most;  // rows of this pass
      const uint32_t off = (done * B + threadIdx.x) * 16;
      // a pass of n rows ends where they do
      const uint32_t end = (done + n) * B < nvec ? (done + n) * B * 16 : nvec * 16;
      auto go = [&](auto split_tag) {
        constexpr bool kSplit = decltype(split_tag)::value;
        const Walk<kSplit ? 0 : CW, BF16, P, kSplit> walk{row, mine, start, W, tl.first, end, splits, inv_w};
        if constexpr (MAXN >= 8 && !(kSplit && CW == 3)) {
          if (n > 4) walk.template rows<8>(off, B * 16);
        }
        if constexpr (MAXN >= 4) {
          if (n > 2 && n <= 4) walk.template rows<4>(off, B * 16);
          if (n == 2) walk.template rows<2>(off, B * 16);
        }
        if (n == 1) walk.column(off);
      };
      if constexpr (kSplits) {
        if (tl.split) go(std::true_type{});
        else go(std::false_type{});
      } else {
        go(std::false_type{});
      }
      done += n;
    }
    // a run that ends a tensor may stop inside a vector: finish it element by element
    const uint32_t rem = tl.n_elems - nvec * VE;
    if (threadIdx.x < rem) {
      const size_t e = size_t(tl.vec_off) * VE + nvec * VE + threadIdx.x;
      // an element behind s boundaries of a split tile starts s workers later
      const uint32_t first = (tl.first + splits.before((nvec * VE + threadIdx.x) * (16 / VE))) % W;
      float acc = -0.0f;
      for (uint32_t k0 = 0; k0 < W; k0 += 8) {
        float x[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) {
          uint32_t w = first + (k0 + i < W ? k0 + i : 0);
          if (w >= W) w -= W;
          if constexpr (BF16) x[i] = widen(reinterpret_cast<gu16_ptr>(row[w])[e]);
          else x[i] = reinterpret_cast<gf32_ptr>(row[w])[e];
        }
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) acc = k0 + i < W ? acc + x[i] : acc;
      }
      if constexpr (BF16) {
        const uint16_t y = uint16_t(bf16_rne(acc * inv_w));
        for (uint32_t k = 0; k < W; ++k) reinterpret_cast<gu16_ptr>(row[k])[e] = y;
      } else {
        const float y = acc * inv_w;
        for (uint32_t k = 0; k < W; ++k) reinterpret_cast<gf32_ptr>(row[k])[e] = y;
      }
    }
  }
}

// Halving-doubling order, one vector per lane, W = 32 or 64: the workers are taken eight at a time:
// their eight vectors are added as a three-level tree, and the partial sums of the blocks are merged
// the way a binary counter carries (block j closes as many levels as j + 1 has trailing zeros), which
// is the same tree  ((x0+x1)+(x2+x3)) + ...  up to its root.
template <bool BF16, int P>
__device__ __forceinline__ void tree_column(const uint64_t* __restrict__ row, uint32_t vec_off, uint32_t W, uint32_t v,
                                            float inv_w) {
  constexpr int kBlk = 8;       // workers per block
  constexpr int kMaxBlocks = 8;  // W <= 64
  const uint32_t n_blocks = W / kBlk;
  Chain<BF16> part[4];  // open partial sums of 8, 16, 32 workers (and the root of 64)
  u32x4 y = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < kMaxBlocks; ++j) {
    if (uint32_t(j) < n_blocks) {
      u32x4 x[kBlk];
#pragma unroll
      for (int i = 0; i < kBlk; ++i)
        x[i] = ld<P>(at(reinterpret_cast<gvec_ptr>(row[j * kBlk + i]) + vec_off, v * 16u));
      __builtin_amdgcn_sched_barrier(0);
      Chain<BF16> t[kBlk];
#pragma unroll
      for (int i = 0; i < kBlk; ++i) t[i].start(x[i]);
#pragma unroll
      for (int s = 1; s < kBlk; s *= 2)
#pragma unroll
        for (int i = 0; i + s < kBlk; i += 2 * s) t[i].merge(t[i + s]);
      // carry: j + 1 = ...1000 closes one level per trailing zero
      int lvl = 0;
#pragma unroll
      for (int m = j + 1; (m & 1) == 0; m >>= 1) {
        part[lvl].merge(t[0]);
        t[0] = part[lvl];
        ++lvl;
      }
      part[lvl] = t[0];
      if (uint32_t(j) + 1 == n_blocks) y = t[0].finish(inv_w);
    }
  }
  for (uint32_t k = 0; k < W; ++k) st<P>(reinterpret_cast<gvec_ptr>(row[k]) + vec_off, v * 16u, y);
}

// The same tree on one element (the ragged end of a tensor).  As many loads at once as tree_column: one
// tile in three of a small job has such an end, and a loop over the blocks that carries its partial sums
// in memory order is felt (64 x 0.3 MiB bf16 25.4 us, 17.5; 32 x 2 MiB 30.6 / 28.5).
template <bool BF16>
__device__ __forceinline__ void tree_element(const uint64_t* __restrict__ row, size_t e, uint32_t W, float inv_w) {
  constexpr int kBlk = 8, kMaxBlocks = 8;
  const uint32_t n_blocks = W / kBlk;
  float part[4];
  float y = 0.f;
#pragma unroll
  for (int j = 0; j < kMaxBlocks; ++j) {
    if (uint32_t(j) < n_blocks) {
      float t[kBlk];
#pragma unroll
      for (int i = 0; i < kBlk; ++i) {
        if constexpr (BF16) t[i] = widen(reinterpret_cast<gu16_ptr>(row[j * kBlk + i])[e]);
        else t[i] = reinterpret_cast<gf32_ptr>(row[j * kBlk + i])[e];
      }
#pragma unroll
      for (int s = 1; s < kBlk; s *= 2)
#pragma unroll
        for (int i = 0; i + s < kBlk; i += 2 * s) t[i] = t[i] + t[i + s];
      int lvl = 0;
#pragma unroll
      for (int m = j + 1; (m & 1) == 0; m >>= 1) {
        t[0] = part[lvl] + t[0];
        ++lvl;
      }
      part[lvl] = t[0];
      if (uint32_t(j) + 1 == n_blocks) y = t[0] * inv_w;
    }
  }
  if constexpr (BF16) {
    const uint16_t o = uint16_t(bf16_rne(y));
    for (uint32_t k = 0; k < W; ++k) reinterpret_cast<gu16_ptr>(row[k])[e] = o;
  } else {
    for (uint32_t k = 0; k < W; ++k) reinterpret_cast<gf32_ptr>(row[k])[e] = y;
  }
}

// W = 32 or 64: small tiles, and whatever is not for k_tree_walk.
template <bool BF16, int P>
__global__ void __launch_bounds__(kMaxBlock)
k_ring_reduce_tree_any(const ReduceTile* __restrict__ tiles, const uint64_t* __restrict__ rows, uint32_t begin,
                       uint32_t count, uint32_t W, float inv_w) {
  constexpr uint32_t VE = BF16 ? 8 : 4;
  for (uint32_t ti = blockIdx.x; ti < count; ti += gridDim.x) {
    const ReduceTile tl = tiles[begin + ti];
    const uint64_t* row = rows + size_t(tl.row) * W;
    const uint32_t nvec = tl.n_elems / VE;
    for (uint32_t v = threadIdx.x; v < nvec; v += blockDim.x) tree_column<BF16, P>(row, tl.vec_off, W, v, inv_w);
    const uint32_t rem = tl.n_elems - nvec * VE;
    if (threadIdx.x < rem)
      tree_element<BF16>(row, size_t(tl.vec_off) * VE + nvec * VE + threadIdx.x, W, inv_w);
  }
}

// Long tiles in the halving-doubling order: the walk of k_walk, replica by replica in bursts, with the
// values added as the balanced tree.  The tree does not depend on the segment, so the workers are read
// in the order 0 .. W-1, two at a time: their sum is merged with the open partial sums the way a binary
// counter carries, which takes log2(W) - 1 partial sums per vector.
//
// Bound: HBM, and how many vectors per lane (bytes per burst) there is room for.  A pair's two bursts
// are issued at once, into two buffers of N vectors; a third buffer, so that the next worker's burst
// flies while a pair is added, measured no faster (VGG-16, 8 workers fp32: 1442 us with, 1408 without;
// ResNet-v2-152, 16 workers: 1239 / 1235).  The partial sums of the highest levels, which change least
// often, lie in LDS where the registers do not hold them all (kLds levels, at most 128 KiB, each lane
// its own slots, so nothing has to be waited for).  That is room for N = 4 (64 KiB per burst) with fp32
// and, up to 16 workers, with bf16, whose sums are twice as large.  Over 32 and 64 workers in bf16 there
// would be room for two vectors, which is slower than small tiles (32 x 33 MiB 449 us, 433; 32 x 70 921 /
// 902; 64 x 70 1843 / 1816; 64 x 100 2662 / 2691): k_ring_reduce_tree_any takes these.  With 36 bytes per lane spilled,
// global loads and two vectors for bf16 before: ResNet-v2-152, 16 workers 1301 -> 1235 us, Transformer
// bf16, 8 workers 2049 -> 1724, ResNet-50, 32 workers fp32 (small tiles only) 1306 -> 1080.
template <int W, bool BF16>
struct TreeShape {
  static constexpr int kLevels = W >= 64 ? 5 : (W >= 32 ? 4 : (W >= 16 ? 3 : (W >= 8 ? 2 : (W >= 4 ? 1 : 0))));
  static constexpr int N = !BF16 && W <= 4 ? 8 : 4;
  static constexpr int kLds = W >= 32 ? 2 : (BF16 && W == 16 ? 1 : 0);
  static constexpr int kSlots = kLds * N * (BF16 ? 2 : 1);  // 16-byte slots per lane
};

// f(0), f(1), ... with each index a constant (a loop pragma gives up on 64 workers)
template <int... I, typename F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// (at most one 1024-lane workgroup per compute unit, like k_walk: 2 x 33 MiB bf16 27.6 -> 25.8 us,
// 8 x 80 MiB fp32 225.3 -> 223.1)
template <int W, bool BF16, int P>
__global__ void __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_tree_walk(const ReduceTile* __restrict__ tiles, const uint64_t* __restrict__ rows, uint32_t begin, uint32_t count,
            uint32_t cap, float inv_w) {
  using S = TreeShape<W, BF16>;
  constexpr uint32_t VE = BF16 ? 8 : 4;
  __shared__ f32x4 high[S::kSlots ? S::kSlots * kMaxBlock : 1];
  for (uint32_t ti = blockIdx.x; ti < count; ti += gridDim.x) {
    const ReduceTile tl = tiles[begin + ti];
    const uint64_t* row = rows + size_t(tl.row) * W;
    const uint32_t nvec = tl.n_elems / VE;
    const uint32_t B = blockDim.x;
    const uint32_t lane = threadIdx.x % 64;
    const uint64_t mine = row[lane < W ? lane : W - 1] + uint64_t(tl.vec_off) * 16;  // kept by lane w for replica w
    const uint32_t total_rows = (nvec + B - 1) / B;
    for (uint32_t done = 0; done < total_rows;) {
      const uint32_t left = total_rows - done;
      const uint32_t n = left < cap ? left : cap;  // rows of this pass
      const uint32_t off = (done * B + threadIdx.x) * 16, stride = B * 16;
      const uint32_t end = (done + n) * B < nvec ? (done + n) * B * 16 : nvec * 16;
      auto res = [&](int w) {
        const uint64_t base = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(mine >> 32), w))) << 32 |
                              uint32_t(__builtin_amdgcn_readlane(int(mine), w));
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base), 0, int(end), kRawBuffer);
      };
      auto pass = [&](auto n_tag) {
        constexpr int N = decltype(n_tag)::value;
        u32x4 buf[2][N];
        Chain<BF16> low[S::kLevels ? S::kLevels : 1][N];  // (the levels that lie in LDS stay unused here)
        u32x4 y[N];
        auto load = [&](int k) {
          const __amdgpu_buffer_rsrc_t r = res(k);
#pragma unroll
          for (int u = 0; u < N; ++u)
            buf[k % 2][u] = __builtin_amdgcn_raw_buffer_load_b128(r, int(off + u * stride), 0, kLoadBits<P>);
        };
        auto slot = [&](int level, int u, int half) -> f32x4& {
          constexpr int kHalves = BF16 ? 2 : 1;
          return high[(((level - (S::kLevels - S::kLds)) * N + u) * kHalves + half) * B + threadIdx.x];
        };
        auto get = [&](int level, int u) {
          if (level < S::kLevels - S::kLds) return low[level][u];
          Chain<BF16> c;
          c.a = slot(level, u, 0);
          if constexpr (BF16) c.b = slot(level, u, 1);
          return c;
        };
        auto put = [&](int level, int u, const Chain<BF16>& c) {
          if (level < S::kLevels - S::kLds) {
            low[level][u] = c;
          } else {
            slot(level, u, 0) = c.a;
            if constexpr (BF16) slot(level, u, 1) = c.b;
          }
        };
        for_each_index(std::make_integer_sequence<int, W / 2>{}, [&](auto pair) {
          constexpr int k = 2 * decltype(pair)::value + 1;
          load(k - 1);
          load(k);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < N; ++u) {
            Chain<BF16> t;
            t.start(buf[0][u]);
            t.add(buf[1][u]);
            constexpr int kClosed = __builtin_ctz(~(k >> 1));  // levels that this pair closes
#pragma unroll
            for (int level = 0; level < kClosed; ++level) {
              Chain<BF16> o = get(level, u);  // the earlier partial sum + the later one
              o.merge(t);
              t = o;
            }
            t.pin();
            if (k + 1 < W) put(kClosed, u, t);
            else y[u] = t.finish(inv_w);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll(W < 16 ? W : 16)
        for (int k = 0; k < W; ++k) {
          const __amdgpu_buffer_rsrc_t r = res(k);
#pragma unroll
          for (int u = 0; u < N; ++u) __builtin_amdgcn_raw_buffer_store_b128(y[u], r, int(off + u * stride), 0, kStoreBits<P>);
        }
      };
      if constexpr (S::N >= 8) {
        if (n > 4) pass(std::integral_constant<int, 8>{});
      }
      if constexpr (S::N >= 4) {
        if (n > 2 && n <= 4) pass(std::integral_constant<int, 4>{});
      }
      if (n == 2) pass(std::integral_constant<int, 2>{});
      if (n == 1) {
        if constexpr (W >= 32) {
          if (off < end) tree_column<BF16, P>(row, tl.vec_off, W, off / 16, inv_w);
        } else {
          u32x4 x[W];
#pragma unroll
          for (int k = 0; k < W; ++k) x[k] = __builtin_amdgcn_raw_buffer_load_b128(res(k), int(off), 0, kLoadBits<P>);
          __builtin_amdgcn_sched_barrier(0);
          const u32x4 y = combine<W, BF16, true>(x, inv_w);
#pragma unroll
          for (int k = 0; k < W; ++k) __builtin_amdgcn_raw_buffer_store_b128(y, res(k), int(off), 0, kStoreBits<P>);
        }
      }
      done += n;
    }
    const uint32_t rem = tl.n_elems - nvec * VE;
    if (threadIdx.x < rem) {
      const size_t e = size_t(tl.vec_off) * VE + nvec * VE + threadIdx.x;
      if constexpr (W >= 32) {
        tree_element<BF16>(row, e, W, inv_w);
      } else {
        float x[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
          if constexpr (BF16) x[k] = widen(reinterpret_cast<gu16_ptr>(row[k])[e]);
          else x[k] = reinterpret_cast<gf32_ptr>(row[k])[e];
        }
        const float y = combine_scalar<W, true>(x, inv_w);
        if constexpr (BF16) {
          const uint16_t o = uint16_t(bf16_rne(y));
#pragma unroll
          for (int k = 0; k < W; ++k) reinterpret_cast<gu16_ptr>(row[k])[e] = o;
        } else {
#pragma unroll
          for (int k = 0; k < W; ++k) reinterpret_cast<gf32_ptr>(row[k])[e] = y;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// pack / unpack: one 1024-lane workgroup per copy tile (at most 1024 vectors of one member, so a
// lane moves one vector and one load instruction of the workgroup covers 16 contiguous KiB),
// grid.y = worker.  A tiny member leaves most lanes idle; measured against one wavefront per 8 KiB
// run, which keeps every lane busy, this is 2 to 7 points of peak faster where it matters and
// equal where the members are small.
template <typename E, bool UNPACK, int P>
__global__ void __launch_bounds__(kCopyBlock)
k_copy(const CopyTile* __restrict__ tiles, const uint64_t* __restrict__ rows, uint32_t begin, uint32_t count,
       uint32_t W, uint32_t fused_row) {
  constexpr uint32_t VE = 16 / sizeof(E);
  const uint32_t lane = threadIdx.x;
  const CopyTile t = tiles[begin + blockIdx.x];
  const uint32_t w = blockIdx.y;
  gvec_ptr tp = reinterpret_cast<gvec_ptr>(rows[size_t(t.row) * W + w]) + t.t_vec_off;
  gvec_ptr fp = reinterpret_cast<gvec_ptr>(rows[size_t(fused_row) * W + w]) + t.f_vec_off;
  const uint32_t nvec = t.n_elems / VE;
  gvec_ptr src = UNPACK ? fp : tp;
  gvec_ptr dst = UNPACK ? tp : fp;
  // (source and destination of a vector share one 64-bit lane offset; a 32-bit one for the stores alone
  // costs two registers and an addition more: small stages 0.6 % slower, 18.03 -> 18.15 us for 4 x 8 MiB)
  for (uint32_t v = lane; v < nvec; v += kCopyBlock) st<P>(dst + v, ld<P>(src + v));
  // ragged end of a member, and (pack only) the +0.0 padding up to the next member
  CARAMEL_GLOBAL E* se = reinterpret_cast<CARAMEL_GLOBAL E*>(src);
  CARAMEL_GLOBAL E* de = reinterpret_cast<CARAMEL_GLOBAL E*>(dst);
  const uint32_t end = UNPACK ? t.n_elems : t.n_elems + t.n_zero;
  for (uint32_t e = nvec * VE + lane; e < end; e += kCopyBlock) de[e] = (e < t.n_elems) ? se[e] : E(0);
}

// ------------------------------------------------------------------------------------------
// Jobs cut into slices (SliceTable; choose_slices() says which).
//
// Bound: HBM, and for the smallest the chain of waits from the table's entries to the values to the stores.  A tile
// costs a workgroup two dependent lookups (tile, base addresses) and belongs to one run; a small job of many runs
// was thousands of such workgroups, which read and write at the same time all over the memory.  A slice's places are
// looked up at once, already in the order in which its workers are added, and a workgroup gets an equal share of
// the job, of whatever runs.  k_slices and k_tree_slices hold N slices per wavefront so that all of a job fits one
// round: everything is read before anything is written.  k_slice and k_tree_slice hold one, with all
// workers' values on the way at once: the smallest jobs, and longer ones in many rounds.
// 8 workers fp32, tiles / slices: 0.25 MiB per replica 4.4 / 3.8 us, 4 MiB 14.6 / 11.4, 16 MiB 51.2 / 47.0 (4.6 -> 5.9 and 5.2 ->
// 5.7 TB/s for the last two), a call of 200 odd tensors of 15 MB 50.4 / 43.5.
//
// The tables are read through the constant address space: scalar loads, also between stores.
typedef const __attribute__((address_space(4))) uint32_t* const_u32_ptr;

// One wavefront's slices: where they lie, how long they are, and how their results go out.
template <bool BF16, int P, int N>
struct Slices {
  const_u32_ptr at, bytes;
  uint64_t base;
  uint32_t W, off;  // off: this lane's vector
  uint32_t len[N], odd;
  __device__ __forceinline__ Slices(const uint32_t* places, const uint32_t* lengths, uint64_t b, uint32_t workers)
      : base(b), W(workers) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) / 64);
    at = (const_u32_ptr)places + size_t(wave) * W * N;
    bytes = (const_u32_ptr)lengths + size_t(wave) * (N + 1);
    off = threadIdx.x % 64 * 16;
#pragma unroll
    for (int u = 0; u < N; ++u) len[u] = bytes[u];
    odd = BF16 ? bytes[N] : 0u;
  }
  // A slice is a buffer of its own length: lanes and dwords beyond it read zeros and store nothing.  (The dword of an
  // odd last bf16 value is read whole; the two bytes behind the value, in the same aligned dword, go nowhere.)
  __device__ __forceinline__ uint64_t address(uint32_t place) const { return base + (uint64_t(place) << 4); }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t res(uint32_t place, uint32_t n) const {
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(address(place)), 0, int(n), kRawBuffer);
  }
  // One word of every line of the places: the steps' lookups miss the caches together and not one by one
  // (first call on new buffers: 8 workers, 16 MiB 64.6 -> 61.3 us, 16 workers 113 -> 107; repeated ones the
  // same).  To be consumed after the last step.
  __device__ __forceinline__ uint32_t touch() const {
    const uint32_t line = threadIdx.x % 64 * 32;
    return reinterpret_cast<gu32_ptr>(reinterpret_cast<uint64_t>(at))[line < W * N ? line : 0];
  }
  // CW: the number of workers, 0 if known at run time only
  template <int CW>
  __device__ __forceinline__ void put(const u32x4 (&y)[N]) {
    if constexpr (BF16) {
#pragma unroll
      for (int u = 0; u < N; ++u) len[u] -= 4 * (odd >> u & 1u);  // whole dwords
    }
#pragma unroll(CW ? CW : 2)
    for (uint32_t k = 0; k < W; ++k)
#pragma unroll
      for (int u = 0; u < N; ++u)
        __builtin_amdgcn_raw_buffer_store_b128(y[u], res(at[k * N + u], len[u]), int(off), 0, kStoreBits<P>);
    if (BF16 && odd) {  // half a dword is left of some slice
#pragma unroll
      for (int u = 0; u < N; ++u)
        if ((odd >> u & 1u) && off == (len[u] & ~15u)) {
          const uint32_t q = (len[u] & 15u) / 4;
          const uint32_t v = q == 0 ? y[u].x : (q == 1 ? y[u].y : (q == 2 ? y[u].z : y[u].w));
#pragma unroll(CW ? CW : 4)
          for (uint32_t k = 0; k < W; ++k) *reinterpret_cast<gu16_ptr>(address(at[k * N + u]) + len[u]) = uint16_t(v);
        }
    }
  }
};

// Chains.  Two buffers: the next worker's N vectors are on the way while a worker's are added (with four, of 512
// registers, nothing was gained from 8 workers on and 5 to 10 % lost with 2 and 3).  256 lanes are one wavefront per
// SIMD: N up to 20 with fp32 sums, 16 with bf16.
template <bool BF16, int P, int N, int LANES>
__global__ void __launch_bounds__(LANES) __attribute__((amdgpu_waves_per_eu(LANES / 256, LANES / 256)))
k_slices(const uint32_t* places, const uint32_t* lengths, uint64_t base, uint32_t W, float inv_w) {
  Slices<BF16, P, N> sl(places, lengths, base, W);
  uint32_t a[N];  // the slices in the next worker, looked up a step ahead
  auto look = [&](uint32_t k) {
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = sl.at[k * N + u];
  };
  Chain<BF16> acc[N];
  u32x4 buf[2][N];
#pragma unroll
  for (int u = 0; u < N; ++u) acc[u].zero();
  auto load = [&](uint32_t k, int j) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      buf[j][u] = __builtin_amdgcn_raw_buffer_load_b128(sl.res(a[u], sl.len[u]), int(sl.off), 0, kLoadBits<P>);
    __builtin_amdgcn_sched_barrier(0);
    look(k + 1 < W ? k + 1 : 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto add = [&](int j) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      acc[u].add(buf[j][u]);
      acc[u].pin();
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  look(0);
  const uint32_t touched = sl.touch();
  load(0, 0);
  uint32_t k = 0;
#pragma unroll 1
  for (; k + 2 < W; k += 2) {
    load(k + 1, 1);
    add(0);
    load(k + 2, 0);
    add(1);
  }
  if (k + 1 < W) load(k + 1, 1);
  add(0);
  if (k + 1 < W) add(1);
  u32x4 y[N];
#pragma unroll
  for (int u = 0; u < N; ++u) y[u] = acc[u].finish(inv_w);
  asm volatile("" ::"v"(touched));
  sl.template put<0>(y);
}

// One slice per wavefront.  CW: the number of workers, 0 if known at run time only.  The values of up to
// kAhead workers are fetched at once.
template <bool BF16, int P, int CW>
__global__ void __launch_bounds__(256)
k_slice(const uint32_t* places, const uint32_t* lengths, uint64_t base, uint32_t workers, float inv_w) {
  const uint32_t W = CW ? uint32_t(CW) : workers;
  Slices<BF16, P, 1> sl(places, lengths, base, W);
  constexpr int kAhead = CW ? CW : 8;
  Chain<BF16> acc;
  acc.zero();
#pragma unroll 1
  for (uint32_t k0 = 0; k0 < W; k0 += kAhead) {
    u32x4 x[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const bool in = (CW && CW % kAhead == 0) || k0 + i < W;
      x[i] = __builtin_amdgcn_raw_buffer_load_b128(sl.res(sl.at[k0 + i], in ? sl.len[0] : 0u), int(sl.off), 0, kLoadBits<P>);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if ((CW && CW % kAhead == 0) || k0 + i < W) acc.add(x[i]);
  }
  const u32x4 y[1] = {acc.finish(inv_w)};
  sl.template put<CW>(y);
}

// Halving-doubling over slices: the workers in the order 0 .. W-1, their sums as the balanced tree
// (as in k_tree_walk).  One round of 256-lane workgroups, like k_slices: one wavefront per SIMD, so 512 registers
// hold four buffers and the open partial sums of every level.  The next pair of workers is on its way while a pair is
// added.  Eight workers to a turn of the loop; the sums of the turns are merged by its number's trailing ones.
// Bound: HBM, and the latencies of W / 2 pairs.  No vector register is spilled, but scalar ones are, to lanes of vector
// registers (N places and as many buffer descriptors of four words): 8 workers none, 2 and 4 workers up to 134, at the
// widest, 16 to 64 workers 6 to 12 with N = 4, 54 to 82 with 6, up to 249 with 14.
template <bool BF16, int P, int W, int N>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_tree_slices(const uint32_t* places, const uint32_t* lengths, uint64_t base, float inv_w) {
  constexpr int kTurn = W < 8 ? W : 8, kTurns = W / kTurn, kPairs = kTurn / 2;
  Slices<BF16, P, N> sl(places, lengths, base, W);
  uint32_t a[N];
  auto look = [&](uint32_t k) {
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = sl.at[k * N + u];
  };
  u32x4 buf[4][N], y[N];
  auto load = [&](uint32_t k, int j) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      buf[j][u] = __builtin_amdgcn_raw_buffer_load_b128(sl.res(a[u], sl.len[u]), int(sl.off), 0, kLoadBits<P>);
    __builtin_amdgcn_sched_barrier(0);
    look(k + 1 < uint32_t(W) ? k + 1 : 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  look(0);
  const uint32_t touched = sl.touch();
  load(0, 0);
  load(1, 1);
  Chain<BF16> low[2][N], high[3][N];  // open sums of 2 and 4 workers; of 8, 16 and 32
#pragma unroll 1
  for (uint32_t turn = 0; turn < uint32_t(kTurns); ++turn) {
#pragma unroll
    for (int p = 0; p < kPairs; ++p) {
      if (p + 1 < kPairs || turn + 1 < uint32_t(kTurns)) {
        load(turn * kTurn + 2 * p + 2, (2 * p + 2) % 4);
        load(turn * kTurn + 2 * p + 3, (2 * p + 3) % 4);
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
        Chain<BF16> t;
        t.start(buf[2 * p % 4][u]);
        t.add(buf[(2 * p + 1) % 4][u]);
        if (p % 2 == 1) {
          low[0][u].merge(t);
          t = low[0][u];
        }
        if (p % 4 == 3) {
          low[1][u].merge(t);
          t = low[1][u];
        }
        t.pin();
        low[p % 4 == 1 && kPairs > 2 ? 1 : 0][u] = t;  // the last pair of a turn leaves the turn's sum in low[0]
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    auto close = [&](int level) {  // the earlier sum + the later one
#pragma unroll
      for (int u = 0; u < N; ++u) {
        high[level][u].merge(low[0][u]);
        low[0][u] = high[level][u];
        low[0][u].pin();
      }
    };
    auto keep = [&](int level) {
#pragma unroll
      for (int u = 0; u < N; ++u) high[level][u] = low[0][u];
    };
    if constexpr (kTurns > 1) {
      if (!(turn & 1)) {
        keep(0);
      } else {
        close(0);
        if constexpr (kTurns > 2) {
          if (!(turn & 2)) {
            keep(1);
          } else {
            close(1);
            if constexpr (kTurns > 4) {
              if (!(turn & 4)) keep(2);
              else close(2);
            }
          }
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < N; ++u) y[u] = low[0][u].finish(inv_w);
  asm volatile("" ::"v"(touched));
  sl.template put<0>(y);
}

// One slice per wavefront, all values at once (eight workers' at a time over 32 and 64).
template <bool BF16, int P, int W>
__global__ void __launch_bounds__(256)
k_tree_slice(const uint32_t* places, const uint32_t* lengths, uint64_t base, float inv_w) {
  Slices<BF16, P, 1> sl(places, lengths, base, W);
  auto fetch = [&](int k) { return __builtin_amdgcn_raw_buffer_load_b128(sl.res(sl.at[k], sl.len[0]), int(sl.off), 0, kLoadBits<P>); };
  u32x4 y[1];
  if constexpr (W <= 16) {
    u32x4 x[W];
#pragma unroll
    for (int k = 0; k < W; ++k) x[k] = fetch(k);
    __builtin_amdgcn_sched_barrier(0);
    y[0] = combine<W, BF16, true>(x, inv_w);
  } else {
    Chain<BF16> part[4];
    for_each_index(std::make_integer_sequence<int, W / 8>{}, [&](auto block) {
      constexpr int j = decltype(block)::value;
      u32x4 x[8];
      Chain<BF16> t[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = fetch(8 * j + i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i].start(x[i]);
#pragma unroll
      for (int s = 1; s < 8; s *= 2)
#pragma unroll
        for (int i = 0; i + s < 8; i += 2 * s) t[i].merge(t[i + s]);
      constexpr int kClosed = __builtin_ctz(~j);
#pragma unroll
      for (int level = 0; level < kClosed; ++level) {
        part[level].merge(t[0]);
        t[0] = part[level];
      }
      if constexpr (j + 1 < W / 8) part[kClosed] = t[0];
      else y[0] = t[0].finish(inv_w);
    });
  }
  sl.template put<W <= 16 ? W : 0>(y);
}

// The table of a job's slices, once per bind: a lane works one slice out for up to kTableSteps workers (place_slice),
// a workgroup as many whole wavefronts' slices as it has lanes for.  Bound: latency, a binary search of log2(pieces)
// dependent loads (4 us with 200 slices, 8 us with 92000, 12 us for 64 workers, 22 without the split of their steps).
// Written by the host and sent, 4 bytes per slice and worker, the table made a bind 1.4 to 4 times as long as one
// with tiles alone, and the call after it up to 5 %: us, bind and first call with tiles, with the host's table, now:
// 8 workers 16 MiB 182 + 70, 313 + 68, 188 + 64; 16 workers 16 MiB 256 + 103, 496 + 107, 268 + 103; 2 workers 90 MiB
// 113 + 82, 453 + 76, 116 + 71; 200 odd tensors of 15 MB apart 217 + 70, 351 + 68, 229 + 63.
constexpr uint32_t kTableBlock = 256, kTableSteps = 16;

__global__ void __launch_bounds__(kTableBlock)
k_slice_table(SliceTable t, const SlicePiece* __restrict__ pieces, const uint64_t* __restrict__ rows,
              uint32_t* __restrict__ places, uint32_t* __restrict__ lengths) {
  __shared__ uint32_t odd[kTableBlock];
  const uint32_t per_block = kTableBlock / t.vecs;  // wavefronts of the job
  const uint32_t mine = threadIdx.x / t.vecs, u = threadIdx.x % t.vecs, wave = blockIdx.x * per_block + mine;
  const uint32_t k0 = blockIdx.y * kTableSteps, k1 = min(k0 + kTableSteps, t.world);
  const bool in = mine < per_block && wave < t.waves();
  uint32_t* const out = lengths + size_t(wave) * (t.vecs + 1);
  odd[threadIdx.x] = 0;
  __syncthreads();
  if (in) {
    const uint32_t len = place_slice(t, pieces, rows, wave, u, k0, k1, places + size_t(wave) * t.world * t.vecs + u);
    if (blockIdx.y == 0) out[u] = (len + 3) & ~3u;
    if (len & 3u) atomicOr(&odd[mine], 1u << u);
  }
  __syncthreads();
  if (in && u == 0 && blockIdx.y == 0) out[t.vecs] = odd[mine];
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 16) places[t.at_words() - 16 + threadIdx.x] = 0;
}

template <int W, int U>
hipError_t launch_w(const ReduceArgs& a, dim3 grid, float inv_w, hipStream_t s) {
#define CARAMEL_GO(BF, P, TR) \
  hipLaunchKernelGGL((k_ring_reduce<W, U, BF, P, TR>), grid, dim3(a.block), 0, s, a.tiles, a.rows, a.begin, a.count, inv_w)
#define CARAMEL_GO2(BF, P) \
  do { if (kTree && a.tree) CARAMEL_GO(BF, P, kTree); else CARAMEL_GO(BF, P, false); } while (0)
  constexpr bool kTree = W > 1;  // a tree over one worker is the chain
  if (a.bf16) {
    if (a.policy != kPlain) CARAMEL_GO2(true, kStream); else CARAMEL_GO2(true, kPlain);
  } else {
    if (a.policy != kPlain) CARAMEL_GO2(false, kStream); else CARAMEL_GO2(false, kPlain);
  }
#undef CARAMEL_GO2
#undef CARAMEL_GO
  return hipGetLastError();
}

template <int W>
hipError_t launch_tree(const ReduceArgs& a, dim3 grid, float inv_w, hipStream_t s) {
#define CARAMEL_TREE(BF, P) \
  hipLaunchKernelGGL((k_tree_walk<W, BF, P>), grid, dim3(a.block), 0, s, a.tiles, a.rows, a.begin, a.count, \
                     a.stream_major < uint32_t(TreeShape<W, BF>::N) ? a.stream_major : uint32_t(TreeShape<W, BF>::N), inv_w)
#define CARAMEL_TREE3(BF) \
  do { \
    if (a.policy == kThrough) CARAMEL_TREE(BF, kThrough); \
    else if (a.policy == kStream) CARAMEL_TREE(BF, kStream); \
    else CARAMEL_TREE(BF, kPlain); \
  } while (0)
  if constexpr (W <= 16)
    if (a.bf16) {
      CARAMEL_TREE3(true);
      return hipGetLastError();
    }
  CARAMEL_TREE3(false);
#undef CARAMEL_TREE3
#undef CARAMEL_TREE
  return hipGetLastError();
}

template <int W>
hipError_t launch_u(const ReduceArgs& a, dim3 grid, float inv_w, hipStream_t s) {
  if constexpr (W > 1)
    if (a.stream_major && a.tree) return launch_tree<W>(a, grid, inv_w, s);
  // W * U vectors per lane must fit the register budget of a 1024-lane workgroup
  constexpr uint32_t kMaxU = W <= 4 ? 4 : (W <= 8 ? 2 : 1);
  uint32_t u = a.unroll ? a.unroll : kMaxU;
  if (u > kMaxU) u = kMaxU;
  if constexpr (kMaxU >= 4) if (u >= 4) return launch_w<W, 4>(a, grid, inv_w, s);
  if constexpr (kMaxU >= 2) if (u >= 2) return launch_w<W, 2>(a, grid, inv_w, s);
  return launch_w<W, 1>(a, grid, inv_w, s);
}

}  // namespace

hipError_t launch_ring_reduce(const ReduceArgs& a, hipStream_t s) {
  if (a.count == 0) return hipSuccess;
  if (a.block != 256 && a.block != 512 && a.block != 1024) return hipErrorInvalidValue;
  uint32_t g = a.count;
  if (a.max_grid && g > a.max_grid) g = a.max_grid;
  const dim3 grid(g);
  const float inv_w = 1.0f / float(a.world);
  const bool tree = a.tree && a.world > 1;  // a tree over one worker is the chain
  // One worker is a plain scaling: small tiles take the kernel that fetches all values at once (4 MiB: 4.3
  // us, 4.8 with the rolled walk's column; 20 MiB 8.1 / 13.3), long ones the unrolled walk (33 MiB fp32
  // 14.6 / 17.2, 260 MiB 85.9 / 90.5; all at once 14.1 and 90.6).
  const bool any = !(a.world == 1 || a.world == 2 || a.world == 4 || a.world == 8 || a.world == 16);
  if (!tree && (a.stream_major || any)) {
#define CARAMEL_WALK(CW, BF, P, MAXN) \
  hipLaunchKernelGGL((k_walk<CW, BF, P, MAXN>), grid, dim3(a.block), 0, s, a.tiles, a.rows, a.begin, a.count, a.world, \
                     a.stream_major < MAXN ? (a.stream_major ? a.stream_major : 1u) : uint32_t(MAXN), inv_w)
#define CARAMEL_WALK3(CW, BF, MAXN) \
  do { \
    if (a.policy == kThrough) CARAMEL_WALK(CW, BF, kThrough, MAXN); \
    else if (a.policy == kStream) CARAMEL_WALK(CW, BF, kStream, MAXN); \
    else CARAMEL_WALK(CW, BF, kPlain, MAXN); \
  } while (0)
#define CARAMEL_WALK_T(CW) \
  do { if (a.bf16) CARAMEL_WALK3(CW, true, 4); else CARAMEL_WALK3(CW, false, 8); } while (0)
    // Three workers: 2 MiB fp32 4.9 us with the rolled walk, 4.3; 3 MiB 5.5 / 4.9; 33 MiB 37.5 / 37.2; 260 MiB
    // equal; but 30 MiB 32.8 / 33.4.
    if (!a.stream_major && a.world == 3) {
      if (a.bf16) CARAMEL_WALK3(3, true, 1); else CARAMEL_WALK3(3, false, 1);
    } else if (!a.stream_major) {
      if (a.bf16) CARAMEL_WALK3(0, true, 1); else CARAMEL_WALK3(0, false, 1);
    } else if (a.world == 1) {
      CARAMEL_WALK_T(1);
    } else if (a.world == 2) {
      CARAMEL_WALK_T(2);
    } else if (a.world == 3) {
      CARAMEL_WALK_T(3);
    } else if (a.world == 4) {
      CARAMEL_WALK_T(4);
    } else if (a.world == 8) {
      CARAMEL_WALK_T(8);
    } else {
      CARAMEL_WALK_T(0);
    }
#undef CARAMEL_WALK_T
#undef CARAMEL_WALK3
#undef CARAMEL_WALK
    return hipGetLastError();
  }
  switch (a.world) {
    case 1: return launch_u<1>(a, grid, inv_w, s);
    case 2: return launch_u<2>(a, grid, inv_w, s);
    case 4: return launch_u<4>(a, grid, inv_w, s);
    case 8: return launch_u<8>(a, grid, inv_w, s);
    case 16: return launch_u<16>(a, grid, inv_w, s);
    default: break;
  }
  if (a.world != 32 && a.world != 64) return hipErrorInvalidValue;
  if (a.stream_major && !a.bf16) return a.world == 32 ? launch_tree<32>(a, grid, inv_w, s) : launch_tree<64>(a, grid, inv_w, s);
#define CARAMEL_TREE(BF, P) \
  hipLaunchKernelGGL((k_ring_reduce_tree_any<BF, P>), grid, dim3(a.block), 0, s, a.tiles, a.rows, a.begin, a.count, a.world, inv_w)
  if (a.bf16) {
    if (a.policy != kPlain) CARAMEL_TREE(true, kStream); else CARAMEL_TREE(true, kPlain);
  } else {
    if (a.policy != kPlain) CARAMEL_TREE(false, kStream); else CARAMEL_TREE(false, kPlain);
  }
#undef CARAMEL_TREE
  return hipGetLastError();
}

hipError_t launch_slice_table(const SliceTable& t, const SlicePiece* pieces, const uint64_t* rows, uint32_t* at,
                              uint32_t* bytes, hipStream_t s) {
  if (t.vecs == 0 || t.vecs > kTableBlock || t.groups == 0) return hipErrorInvalidValue;
  const uint32_t per_block = kTableBlock / t.vecs;
  hipLaunchKernelGGL(k_slice_table, dim3((t.waves() + per_block - 1) / per_block, (t.world + kTableSteps - 1) / kTableSteps),
                     dim3(kTableBlock), 0, s, t, pieces, rows, at, bytes);
  return hipGetLastError();
}

hipError_t launch_slices(const SliceArgs& a, hipStream_t s) {
  const float inv_w = 1.0f / float(a.world);
  const dim3 grid(a.groups), lanes(a.lanes);
  const bool through = a.policy == kThrough;
#define CARAMEL_SKIP(...)
#define CARAMEL_ROUND(BF, TH, N, L) \
  if (a.vecs == N && a.bf16 == BF && through == TH && a.lanes == L) { \
    hipLaunchKernelGGL((k_slices<BF, TH ? kThrough : kStream, N, L>), grid, lanes, 0, s, a.at, a.bytes, a.base, a.world, inv_w); \
    return hipGetLastError(); \
  }
#define CARAMEL_ONE(BF, TH, CW) \
  if ((CW == 0 || a.world == CW) && a.bf16 == BF && through == TH) { \
    hipLaunchKernelGGL((k_slice<BF, TH ? kThrough : kStream, CW>), grid, lanes, 0, s, a.at, a.bytes, a.base, a.world, inv_w); \
    return hipGetLastError(); \
  }
#define CARAMEL_TREE_ROUND(W, BF, N) \
  if (a.vecs == N && a.world == W && a.bf16 == BF && !through && a.lanes == 256) { \
    hipLaunchKernelGGL((k_tree_slices<BF, kStream, W, N>), grid, lanes, 0, s, a.at, a.bytes, a.base, inv_w); \
    return hipGetLastError(); \
  }
#define CARAMEL_TREE_ONE(W, BF, TH) \
  if (a.world == W && a.bf16 == BF && through == TH) { \
    hipLaunchKernelGGL((k_tree_slice<BF, TH ? kThrough : kStream, W>), grid, lanes, 0, s, a.at, a.bytes, a.base, inv_w); \
    return hipGetLastError(); \
  }
  if (a.vecs == 1 && a.lanes == 256) {
    if (a.tree) {
      CARAMEL_SLICE_KERNELS(CARAMEL_SKIP, CARAMEL_SKIP, CARAMEL_SKIP, CARAMEL_TREE_ONE)
    } else {
      CARAMEL_SLICE_KERNELS(CARAMEL_SKIP, CARAMEL_ONE, CARAMEL_SKIP, CARAMEL_SKIP)
    }
  } else if (a.tree) {
    CARAMEL_SLICE_KERNELS(CARAMEL_SKIP, CARAMEL_SKIP, CARAMEL_TREE_ROUND, CARAMEL_SKIP)
  } else {
    CARAMEL_SLICE_KERNELS(CARAMEL_ROUND, CARAMEL_SKIP, CARAMEL_SKIP, CARAMEL_SKIP)
  }
#undef CARAMEL_SKIP
#undef CARAMEL_ROUND
#undef CARAMEL_ONE
#undef CARAMEL_TREE_ROUND
#undef CARAMEL_TREE_ONE
  return hipErrorInvalidValue;
}

hipError_t launch_copy(const CopyArgs& a, hipStream_t s) {
  if (a.count == 0) return hipSuccess;
  const dim3 grid(a.count, a.world);
#define CARAMEL_CP(E, UN) \
  do { \
    if (a.policy != kPlain) \
      hipLaunchKernelGGL((k_copy<E, UN, kStream>), grid, dim3(kCopyBlock), 0, s, a.tiles, a.rows, a.begin, a.count, a.world, a.fused_row); \
    else \
      hipLaunchKernelGGL((k_copy<E, UN, kPlain>), grid, dim3(kCopyBlock), 0, s, a.tiles, a.rows, a.begin, a.count, a.world, a.fused_row); \
  } while (0)
  if (a.bf16) {
    if (a.unpack) CARAMEL_CP(uint16_t, true); else CARAMEL_CP(uint16_t, false);
  } else {
    if (a.unpack) CARAMEL_CP(uint32_t, true); else CARAMEL_CP(uint32_t, false);
  }
#undef CARAMEL_CP
  return hipGetLastError();
}

}  // namespace caramel
