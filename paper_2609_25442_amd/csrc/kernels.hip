// gfx950 kernels of the packing and assembly steps (WeightBridge Sec. 3.2:
// a packing kernel coalesces a round's tensors into per-receiver buffers in
// checkpoint format; an assembly kernel scatters them into the inference
// tensors). Both are batched across tensors: one launch walks a flat table of
// work items, each spread over one or more workgroups.
//
//  * wb_tasks_kernel  -- copy/cast work items: 16-byte vectorised row copies,
//    fp32 -> bf16 (v_cvt_pk_bf16_f32, round to nearest even), bf16 -> fp32,
//    rows at any element address and width, an element-wise fallback for rows
//    narrower than a vector, and tiles transposed in registers (below their
//    size through LDS) where a trainer stores a shard transposed. Work
//    items are spread over several one-wave workgroups: a vector kind takes
//    one per chunk of kChunkVecs vectors, each issuing all of its loads, then
//    all of its stores, and exiting (no loop, so no wait on the completion of
//    earlier stores before the next loads, which caps a looping copy well
//    below the rate of these one-shot workgroups on gfx950); a transpose
//    takes one per 64 x 64 (registers) or 32 x 32 (LDS) tile.
//  * wb_qblock_kernel -- fp8 E4M3FN blocks (<= 128 x 128): two single-piece
//    bf16 blocks per workgroup (a row of the pair is one 512-byte load span),
//    other blocks one per workgroup, gathered from their wire pieces; blocks
//    held in registers, amax by wavefront shuffles plus LDS across the four
//    waves, s = amax / 448 (IEEE division),
//    q = RN(x / s) computed with one reciprocal per block and a remainder
//    correction for bf16 sources (exact in the range that reaches E4M3;
//    checked for every bf16 input pair), two for fp32 ones, IEEE division
//    outside those forms' range, then v_cvt_pk_fp8_f32. The scale is written
//    by thread 0.
// The work is bandwidth bound: no matrix cores are involved.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "wb_internal.hpp"

namespace wb {
namespace {

// Tuning knobs (build-time): whether loads / stores carry the non-temporal
// hint (every byte is touched once), and dynamic LDS reserved per copy
// workgroup (a cap on workgroups per CU). The chunk size is in wb_internal.hpp.
#ifndef WB_NT_LOAD
#define WB_NT_LOAD 1
#endif
#ifndef WB_NT_STORE
#define WB_NT_STORE 1
#endif
#ifndef WB_TASK_DYN_LDS
#define WB_TASK_DYN_LDS 0
#endif
// The fp8 block kernel reserves dynamic LDS to cap the workgroups per CU: two
// (64 KiB) where most blocks go in pairs, three (48 KiB) where most go one per
// workgroup. Three against two for pairs: 1.5 % slower on 2048 and 4096
// column rows (0.45 and 0.53 ms launches), 0.5 % faster on 7168; for single
// fp32 blocks 5.5 % faster (whole unpack 2.06 -> 1.95 ms), four no more (1.94
// and 1.94 ms).
constexpr unsigned kQBlockLdsPairs = 65536, kQBlockLdsSingles = 49152;

constexpr int kThreads = kChunkThreads;

template <class T>
__device__ __forceinline__ T ld(const T* p) {
#if WB_NT_LOAD
  return __builtin_nontemporal_load(p);
#else
  return *p;
#endif
}
template <class T>
__device__ __forceinline__ void st(T v, T* p) {
#if WB_NT_STORE
  __builtin_nontemporal_store(v, p);
#else
  *p = v;
#endif
}

// A table's address as a pointer to global memory, so that accesses through
// it need no check for the LDS aperture (flat instructions).
__device__ __forceinline__ char* global_ptr(uint64_t p) {
  return (char*)reinterpret_cast<__attribute__((address_space(1))) char*>(p);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const bf16x2 h = __builtin_convertvector(f32x2{a, b}, bf16x2);
  return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Walks the flattened (row, vector) index space of a rows x vpr block with
// stride kThreads, keeping row and column incrementally (one division per task).
struct Walker {
  uint32_t r, c, dr, dc, vpr;
  __device__ Walker(uint32_t start, uint32_t vpr_) : vpr(vpr_) {
    r = start / vpr;
    c = start % vpr;
    dr = kThreads / vpr;
    dc = kThreads % vpr;
  }
  __device__ __forceinline__ void step() {
    c += dc;
    r += dr;
    if (c >= vpr) {
      c -= vpr;
      ++r;
    }
  }
};

// Units [q0, q1) of a rows x vpr block in row-major order: lane l takes
// q0 + l + k * kThreads for k < N; on[k] says whether that unit exists.
template <int N = kChunkPerLane>
struct ChunkWalk {
  uint32_t r[N], c[N];
  bool on[N];
  __device__ ChunkWalk(uint32_t q0, uint32_t q1, uint32_t vpr) {
    Walker w(q0 + threadIdx.x, vpr);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      on[k] = q0 + threadIdx.x + k * kThreads < q1;
      r[k] = w.r;
      c[k] = w.c;
      w.step();
    }
  }
};

// 16-byte row copy of one chunk; cols, strides and offsets in bytes.
__device__ void run_copy16(const Task& t, const char* src, char* dst, uint32_t q0) {
  const uint32_t vpr = t.cols >> 4;
  const uint32_t total = t.rows * vpr;
  if (q0 >= total) return;
  const uint32_t q1 = min(total, q0 + uint32_t(kChunkVecs));
  u32x4 v[kChunkPerLane];
  if (t.rows == 1) {
    const u32x4* s = reinterpret_cast<const u32x4*>(src) + q0 + threadIdx.x;
    u32x4* d = reinterpret_cast<u32x4*>(dst) + q0 + threadIdx.x;
    const uint32_t m = q1 - q0;
#pragma unroll
    for (int k = 0; k < kChunkPerLane; ++k)
      if (threadIdx.x + k * kThreads < m) v[k] = ld(s + k * kThreads);
#pragma unroll
    for (int k = 0; k < kChunkPerLane; ++k)
      if (threadIdx.x + k * kThreads < m) st(v[k], d + k * kThreads);
    return;
  }
  const ChunkWalk<> w(q0, q1, vpr);
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k)
    if (w.on[k]) v[k] = ld(reinterpret_cast<const u32x4*>(src + uint64_t(w.r[k]) * t.src_ld) + w.c[k]);
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k)
    if (w.on[k]) st(v[k], reinterpret_cast<u32x4*>(dst + uint64_t(w.r[k]) * t.dst_ld) + w.c[k]);
}

// fp32 -> bf16 of one chunk of 2 kThreads units of 4 elements (chunk c starts
// at unit 2 c kThreads): lane l converts units l and l + kThreads, so each load
// instruction of the wave reads 64 consecutive 16-byte vectors of a row; two
// 8-byte stores. Strides in elements.
__device__ void run_f32_bf16(const Task& t, const char* src, char* dst, uint32_t chunk) {
  const uint32_t vpr = t.cols >> 2;
  const uint32_t total = t.rows * vpr;
  const uint32_t q0 = chunk * 2 * uint32_t(kThreads);
  if (q0 >= total) return;
  const uint32_t q1 = min(total, q0 + 2 * uint32_t(kThreads));
  f32x4 a[2];
  if (t.rows == 1) {  // one run: unit q is input vector q and output half q
    const f32x4* s = reinterpret_cast<const f32x4*>(src) + q0 + threadIdx.x;
    u32x2* d = reinterpret_cast<u32x2*>(dst) + q0 + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (q0 + threadIdx.x + k * kThreads < q1) a[k] = ld(s + k * kThreads);
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (q0 + threadIdx.x + k * kThreads < q1)
        st(u32x2{pack_bf16x2(a[k].x, a[k].y), pack_bf16x2(a[k].z, a[k].w)}, d + k * kThreads);
    return;
  }
  const ChunkWalk<2> w(q0, q1, vpr);
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (w.on[k])
      a[k] = ld(reinterpret_cast<const f32x4*>(src + (uint64_t(w.r[k]) * t.src_ld + uint64_t(w.c[k]) * 4) * 4));
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (w.on[k])
      st(u32x2{pack_bf16x2(a[k].x, a[k].y), pack_bf16x2(a[k].z, a[k].w)},
         reinterpret_cast<u32x2*>(dst + (uint64_t(w.r[k]) * t.dst_ld + uint64_t(w.c[k]) * 4) * 2));
}

// bf16 -> fp32 of one chunk of input vectors (8 elements each); strides in
// elements.
__device__ void run_bf16_f32(const Task& t, const char* src, char* dst, uint32_t q0) {
  const uint32_t vpr = t.cols >> 3;
  const uint32_t total = t.rows * vpr;
  if (q0 >= total) return;
  const uint32_t q1 = min(total, q0 + uint32_t(kChunkVecs));
  u32x4 v[kChunkPerLane];
  if (t.rows == 1) {  // one run: input vector q becomes output vectors 2q and 2q + 1
    const u32x4* s = reinterpret_cast<const u32x4*>(src) + q0 + threadIdx.x;
    f32x4* d = reinterpret_cast<f32x4*>(dst) + 2 * (q0 + threadIdx.x);
#pragma unroll
    for (int k = 0; k < kChunkPerLane; ++k)
      if (q0 + threadIdx.x + k * kThreads < q1) v[k] = ld(s + k * kThreads);
#pragma unroll
    for (int k = 0; k < kChunkPerLane; ++k)
      if (q0 + threadIdx.x + k * kThreads < q1) {
        const u32x4 x = v[k];
        st(f32x4{bf16_lo(x.x), bf16_hi(x.x), bf16_lo(x.y), bf16_hi(x.y)}, d + 2 * k * kThreads);
        st(f32x4{bf16_lo(x.z), bf16_hi(x.z), bf16_lo(x.w), bf16_hi(x.w)}, d + 2 * k * kThreads + 1);
      }
    return;
  }
  const ChunkWalk<> w(q0, q1, vpr);
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k)
    if (w.on[k])
      v[k] = ld(reinterpret_cast<const u32x4*>(src + (uint64_t(w.r[k]) * t.src_ld + uint64_t(w.c[k]) * 8) * 2));
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k)
    if (w.on[k]) {
      const u32x4 x = v[k];
      f32x4* dp = reinterpret_cast<f32x4*>(dst + (uint64_t(w.r[k]) * t.dst_ld + uint64_t(w.c[k]) * 8) * 4);
      st(f32x4{bf16_lo(x.x), bf16_hi(x.x), bf16_lo(x.y), bf16_hi(x.y)}, dp);
      st(f32x4{bf16_lo(x.z), bf16_hi(x.z), bf16_lo(x.w), bf16_hi(x.w)}, dp + 1);
    }
}

// Vectors at element alignment: gfx950 loads and stores global memory at any
// byte address, so an unaligned vector costs the same instruction. A pointer's
// alignment does not survive template deduction (ld and st would promise the
// plain type's), so the type is named here, and the address space with it: a
// flat access would be split.
template <typename T, int kAlign>
struct Unaligned {
  typedef T type __attribute__((aligned(kAlign)));
  typedef __attribute__((address_space(1))) type* ptr;
  typedef const __attribute__((address_space(1))) type* const_ptr;
};

template <typename T, int kAlign, bool kNt = WB_NT_LOAD != 0>
__device__ __forceinline__ T ld_at(const char* p) {
  const auto q = (typename Unaligned<T, kAlign>::const_ptr)(reinterpret_cast<uintptr_t>(p));
  if (kNt) return __builtin_nontemporal_load(q);
  return *q;
}

template <typename T, int kAlign, bool kNt = WB_NT_STORE != 0, typename P>
__device__ __forceinline__ void st_at(T v, P* p) {
  const auto q = (typename Unaligned<T, kAlign>::ptr)(reinterpret_cast<uintptr_t>(p));
  if (kNt)
    __builtin_nontemporal_store(v, q);
  else
    *q = v;
}

// One chunk of a rectangle whose rows sit at any element address (flat shards
// that start anywhere, odd widths): kSs, kDs the element bytes of both sides.
// Lane l of chunk c takes unit 64 c + l: one load and one store; inner units
// are aligned in the destination, and a row's first and last unit overlap
// their neighbours, so no row has single elements. Bound: HBM. A bf16 flat
// shard of a sixth of a 16-layer model (3.2 GB moved), every run at an odd
// phase: 1974 us element by element, 487 us so (6.6 TB/s, the aligned copy's
// rate is 6.7); fp32 -> bf16 at widths 1500 and 1721 (0.9 GB): 771 -> 157 us,
// and 151 with the runs that the planner sends as vectors. Two units per lane:
// 503 and 161 us.
template <int kSs, int kDs>
__device__ __forceinline__ void run_rows(const Task& t, const char* src, char* dst, uint32_t chunk) {
  constexpr int V = 16 / (kSs > kDs ? kSs : kDs);
  const uint32_t q = chunk * uint32_t(kThreads) + threadIdx.x;
  if (q >= t.rows * t.units) return;
  const uint32_t r = t.rows == 1 ? 0 : q / t.units;
  char* dr = dst + uint64_t(r) * t.dst_ld * kDs;
  const int a = int((0u - uint32_t(reinterpret_cast<uintptr_t>(dr))) & uint32_t(V * kDs - 1)) / kDs;
  const int64_t at = int64_t(q - r * t.units) * V + (a ? a - V : 0);
  if (at >= int64_t(t.cols)) return;
  const int64_t off = at < 0 ? 0 : at > int64_t(t.cols) - V ? int64_t(t.cols) - V : at;
  const char* s = src + (uint64_t(r) * t.src_ld + off) * kSs;
  char* d = dr + off * kDs;
  if (kSs == 2 && kDs == 4) {
    const u32x2 x = ld_at<u32x2, 2>(s);
    st_at<u32x4, 2>(u32x4{x.x << 16, x.x & 0xFFFF0000u, x.y << 16, x.y & 0xFFFF0000u}, d);
    return;
  }
  const u32x4 x = ld_at<u32x4, 2>(s);
  if (kSs == 4 && kDs == 2) {
    const f32x4 f = __builtin_bit_cast(f32x4, x);
    st_at<u32x2, 2>(u32x2{pack_bf16x2(f.x, f.y), pack_bf16x2(f.z, f.w)}, d);
  } else {
    st_at<u32x4, 2>(x, d);
  }
}

__device__ void run_rows_any(const Task& t, const char* src, char* dst, uint32_t chunk) {
  if (t.sdt == WB_F32)
    t.ddt == WB_F32 ? run_rows<4, 4>(t, src, dst, chunk) : run_rows<4, 2>(t, src, dst, chunk);
  else
    t.ddt == WB_F32 ? run_rows<2, 4>(t, src, dst, chunk) : run_rows<2, 2>(t, src, dst, chunk);
}

// Raw bits of one element, widened to 32 bits.
__device__ __forceinline__ uint32_t load_bits(const char* p, int dt) {
  if (dt == WB_F32) return *reinterpret_cast<const uint32_t*>(p);
  if (dt == WB_BF16) return *reinterpret_cast<const uint16_t*>(p);
  return *reinterpret_cast<const uint8_t*>(p);
}

__device__ __forceinline__ void store_converted(char* p, uint32_t bits, int sdt, int ddt) {
  if (ddt == WB_F32) {
    *reinterpret_cast<uint32_t*>(p) = sdt == WB_BF16 ? bits << 16 : bits;
  } else if (ddt == WB_BF16) {
    const uint32_t w = sdt == WB_F32 ? pack_bf16x2(__uint_as_float(bits), 0.0f) : bits;
    *reinterpret_cast<uint16_t*>(p) = static_cast<uint16_t>(w);
  } else {
    *reinterpret_cast<uint8_t*>(p) = static_cast<uint8_t>(bits);
  }
}

__device__ __forceinline__ int dt_bytes(int dt) { return dt == WB_F32 ? 4 : (dt == WB_BF16 ? 2 : 1); }

// Element by element; strides in elements.
__device__ void run_scalar(const Task& t, const char* src, char* dst) {
  const int ss = dt_bytes(t.sdt), ds = dt_bytes(t.ddt);
  const uint64_t total = uint64_t(t.rows) * t.cols;
  Walker w(threadIdx.x, t.cols);
  for (uint64_t q = threadIdx.x; q < total; q += kThreads) {
    const uint32_t bits = load_bits(src + (uint64_t(w.r) * t.src_ld + w.c) * ss, t.sdt);
    store_converted(dst + (uint64_t(w.r) * t.dst_ld + w.c) * ds, bits, t.sdt, t.ddt);
    w.step();
  }
}

// dst[c][r] = cvt(src[r][c]) for quarter `part` (32 x 32) of a tile of up to
// 64 x 64, through LDS (padded rows: conflict-free column reads).
__device__ void run_transpose(const Task& t, const char* src, char* dst, uint32_t part) {
  __shared__ uint32_t tile[32][33];
  const uint32_t r0 = (part >> 1) * 32, c0 = (part & 1) * 32;
  if (r0 >= t.rows || c0 >= t.cols) return;  // uniform over the workgroup
  const int ss = dt_bytes(t.sdt), ds = dt_bytes(t.ddt);
  const uint32_t R = min(32u, t.rows - r0), C = min(32u, t.cols - c0);
  src += (uint64_t(r0) * t.src_ld + c0) * ss;
  dst += (uint64_t(c0) * t.dst_ld + r0) * ds;
  for (uint32_t i = threadIdx.x; i < 32 * 32; i += kThreads) {
    const uint32_t r = i >> 5, c = i & 31;
    if (r < R && c < C) tile[r][c] = load_bits(src + (uint64_t(r) * t.src_ld + c) * ss, t.sdt);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < 32 * 32; i += kThreads) {
    const uint32_t c = i >> 5, r = i & 31;
    if (r < R && c < C) store_converted(dst + (uint64_t(c) * t.dst_ld + r) * ds, tile[r][c], t.sdt, t.ddt);
  }
}

// Column j of an 8 x 8 block of 2-byte elements held as eight 16-byte rows.
__device__ __forceinline__ u32x4 column8(const u32x4 (&a)[8], int j) {
  uint32_t o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t x = a[2 * k][j >> 1], y = a[2 * k + 1][j >> 1];
    o[k] = (j & 1) ? ((x >> 16) | (y & 0xFFFF0000u)) : ((x & 0xFFFFu) | (y << 16));
  }
  return u32x4{o[0], o[1], o[2], o[3]};
}

// dst[c][r] = src[r][c] for 2-byte elements, (64..256) rows x 64 columns: each
// wave takes one 64 x 64 tile (tile `w` of the item, counted down the rows),
// each lane an 8 x 8 sub-tile that it loads as eight 16-byte rows, transposes
// in registers and stores as eight 16-byte rows, at any element address on
// both sides. Lanes 8i..8i+7 cover one 128-byte span of a row on both sides.
// Spans that are no whole lines share lines with their neighbours', so the
// stores carry no non-temporal hint (the parts of a line meet in the L2), and
// the loads only where the spans are whole (kNt): with it, 4 transposes of 4097
// x 4099 took 146 (bf16), 292 (fp32), 203 (fp32 -> bf16) and 256 us (bf16 ->
// fp32) against 128, 200, 157 and 186 through LDS tiles without; now 85, 203,
// 131 and 157. Whole spans (4096 x 4096, fp32 -> bf16): 79, 137 through LDS, 95
// with plain loads.
template <bool kNt>
__device__ __forceinline__ void run_transpose16(const Task& t, const char* src, char* dst, uint32_t w) {
  const uint32_t l = threadIdx.x & 63;
  if (w * 64 >= t.rows) return;
  const uint32_t c0 = 8 * (l & 7), r0 = w * 64 + 8 * (l >> 3);
  u32x4 a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    a[i] = ld_at<u32x4, 2, kNt>(src + (uint64_t(r0 + i) * t.src_ld + c0) * 2);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    st_at<u32x4, 2, false>(column8(a, j), dst + (uint64_t(c0 + j) * t.dst_ld + r0) * 2);
}

// dst[c][r] = cvt(src[r][c]) with fp32 on at least one side, (32..128) rows x
// 32 columns: the same with 4 x 4 sub-tiles and 32 x 32 tiles, a 16-byte row
// of a sub-tile on each fp32 side and an 8-byte one on a bf16 side.
template <int kSs, int kDs, bool kNt>
__device__ __forceinline__ void run_transpose4(const Task& t, const char* src, char* dst, uint32_t w) {
  const uint32_t l = threadIdx.x & 63;
  if (w * 32 >= t.rows) return;
  const uint32_t c0 = 4 * (l & 7), r0 = w * 32 + 4 * (l >> 3);
  u32x4 a[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const char* p = src + (uint64_t(r0 + i) * t.src_ld + c0) * kSs;
    if (kSs == 4) {
      a[i] = ld_at<u32x4, 2, kNt>(p);
    } else {
      const u32x2 x = ld_at<u32x2, 2, kNt>(p);
      a[i] = u32x4{x.x << 16, x.x & 0xFFFF0000u, x.y << 16, x.y & 0xFFFF0000u};
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    char* p = dst + (uint64_t(c0 + j) * t.dst_ld + r0) * kDs;
    if (kDs == 4) {
      st_at<u32x4, 2, false>(u32x4{a[0][j], a[1][j], a[2][j], a[3][j]}, p);
    } else {
      st_at<u32x2, 2, false>(u32x2{pack_bf16x2(__uint_as_float(a[0][j]), __uint_as_float(a[1][j])),
                                   pack_bf16x2(__uint_as_float(a[2][j]), __uint_as_float(a[3][j]))},
                             p);
    }
  }
}

template <bool kNt>
__device__ __forceinline__ void run_transpose4_any(const Task& t, const char* src, char* dst, uint32_t w) {
  if (t.sdt == WB_F32)
    t.ddt == WB_F32 ? run_transpose4<4, 4, kNt>(t, src, dst, w) : run_transpose4<4, 2, kNt>(t, src, dst, w);
  else
    run_transpose4<2, 4, kNt>(t, src, dst, w);
}

// Register transposes: w is the tile of the item. A tile's spans of the source
// are whole lines (or aligned halves) where the item's first and its pitch are
// multiples of their size.
__device__ void run_register_transpose(const Task& t, const char* src, char* dst, uint32_t w) {
  const int ss = dt_bytes(t.sdt);
  const uint32_t span = uint32_t(t.cols) * ss;  // 64 or 128 bytes
  const bool whole = ((uint32_t(reinterpret_cast<uintptr_t>(src)) | t.src_ld * uint32_t(ss)) & (span - 1)) == 0;
  if (t.kind == TASK_TRANSPOSE16)
    whole ? run_transpose16<WB_NT_LOAD != 0>(t, src, dst, w) : run_transpose16<false>(t, src, dst, w);
  else
    whole ? run_transpose4_any<WB_NT_LOAD != 0>(t, src, dst, w) : run_transpose4_any<false>(t, src, dst, w);
}

}  // namespace

__device__ __forceinline__ const char* base_of(uint16_t idx, const uint64_t* ptrs, const char* buf, const char* aux) {
  return idx == 0 ? buf : idx == kAuxBuffer ? aux : global_ptr(ptrs[idx]);
}

// XCD-aware order of a launch's work. The hardware hands workgroup b to XCD
// b mod 8 (round-robin over the 8 XCDs), and over a long launch the XCDs drift
// apart, so neighbouring work units (the same DRAM pages; for fp8 blocks, the
// same 128 rows of a wire payload) end up in flight at different times on
// different XCDs. Renumbered so that in each run of 8 C workgroups XCD x takes
// C consecutive units, neighbours are in flight together on one XCD, while the
// eight XCDs still work within one run (so every HBM channel stays busy). A
// bijection of [0, total); a tail shorter than 8 C keeps the plain order.
constexpr uint64_t kXcds = 8;
constexpr uint64_t kXcdRunCopy = 1024;  // copy/cast chunks (1-2 KiB of source each)
constexpr uint64_t kXcdRunPairs = 512;  // fp8 block pairs (64 KiB of wire each)
__device__ __forceinline__ uint64_t xcd_order(uint64_t b, uint64_t total, uint64_t C) {
  const uint64_t run = kXcds * C, base = b / run * run;
  if (base + run > total) return b;
  const uint64_t k = b - base;
  return base + (k % kXcds) * C + k / kXcds;
}

// Workgroups are laid out class by class: item i of class 0 takes workgroups
// [i, i + 1) * 2^s0, chunk = b mod 2^s0 (b in XCD-aware order); then class 1
// the same with s1; then one workgroup per class-2 item. A grid wider than
// kMaxGridX workgroups is folded into rows of gridDim.x.
__global__ __launch_bounds__(kThreads) void wb_tasks_kernel(const Task* __restrict__ tasks,
                                                            const uint64_t* __restrict__ ptrs, const char* buf,
                                                            const char* aux, uint32_t ntasks, uint32_t n0,
                                                            uint32_t n1, uint32_t s0, uint32_t s1) {
  uint64_t b = uint64_t(blockIdx.y) * gridDim.x + blockIdx.x;
  const uint64_t w0 = uint64_t(n0) << s0, w1 = uint64_t(n1) << s1;
  uint64_t ti;
  uint32_t chunk = 0;
  if (b < w0) {
    b = xcd_order(b, w0, kXcdRunCopy);
    ti = b >> s0;
    chunk = uint32_t(b) & ((1u << s0) - 1u);
  } else if ((b -= w0) < w1) {
    ti = n0 + (b >> s1);
    chunk = uint32_t(b) & ((1u << s1) - 1u);
  } else {
    ti = uint64_t(n0) + n1 + (b - w1);
  }
  if (ti >= ntasks) return;
  const Task t = tasks[ti];
  const char* src = base_of(t.src_idx, ptrs, buf, aux) + t.src_off;
  char* dst = const_cast<char*>(base_of(t.dst_idx, ptrs, buf, aux)) + t.dst_off;
  const uint32_t q0 = chunk * uint32_t(kChunkVecs);
  switch (t.kind) {
    case TASK_COPY16: run_copy16(t, src, dst, q0); break;
    case TASK_F32_BF16: run_f32_bf16(t, src, dst, chunk); break;
    case TASK_BF16_F32: run_bf16_f32(t, src, dst, q0); break;
    case TASK_ROWS: run_rows_any(t, src, dst, chunk); break;
    case TASK_SCALAR: if (chunk == 0) run_scalar(t, src, dst); break;
    case TASK_TRANSPOSE: run_transpose(t, src, dst, chunk); break;
    case TASK_TRANSPOSE16:
    case TASK_TRANSPOSE4:
      run_register_transpose(t, src, dst, chunk * (kThreads / 64) + (threadIdx.x >> 6));
      break;
    default: break;
  }
}

// dst[c][r] = src[r][c] of one tile per workgroup (TASK_TILE items): kTileRows x
// kTileCols 2-byte elements, or kTileRows x kTileCols / 2 4-byte ones. Thread t
// takes the 16-byte words at source rows 8 (t / 64) .. + 7, word t mod 64 (a
// wave instruction reads 1 KiB of one source row), and transposes them in
// registers: an 8 x 8 sub-tile of 2-byte elements, two 4 x 4 ones of 4-byte.
// LDS regroups the sub-tiles by destination row, and each thread then stores
// eight 16-byte pieces of destination rows (a wave instruction writes four
// whole 256-byte rows, or two of 512 bytes). Word w of destination row r sits
// in LDS at w ^ ((r / 8) mod 16), or w ^ ((r / 4) mod 32): the sub-tiles of one
// wave land in different banks, and a row read back is a permutation of its
// own words. Bound: HBM, one workgroup (16 waves) per CU by its LDS. 4-byte
// tiles took the fp32 pack of a TP4 rank of half an 8 B dense model (2.4 of
// its 9.1 GB transposed) from 1.64 (LDS tiles of 32 x 32) to 1.42 ms (6.4 TB/s).
// Launches of few 4-byte tiles (kPlainTiles, 256 MiB read and written) go without
// the non-temporal hint: their data may be in the 256 MB cache, where the hint
// cost a quarter (8 x 1000 x 4096: 71 us with it, 53 without; LDS tiles of 32 x
// 32, which these replaced, 50-72). Larger launches are 4 % faster with it (24 x
// 4096 x 4096: 533 and 553).
constexpr uint32_t kPlainTiles = 1024;

template <int kEs, bool kNt>
__device__ __forceinline__ void run_tile(const Task& t, const char* src, char* dst, u32x4* lds) {
  constexpr int V = 16 / kEs, GC = kTileCols * 2 / 16;  // elements per word, words per source row
  constexpr int GR = kTileRows / V, H = 8 / V;          // words per destination row, words a thread gives each
  const int cg = threadIdx.x % GC, rg = threadIdx.x / GC;
  const auto fetch = [](const u32x4* p) { return kNt ? ld(p) : *p; };
  u32x4 a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    a[i] = fetch(reinterpret_cast<const u32x4*>(src + (uint64_t(8 * rg + i) * t.src_ld + V * cg) * kEs));
#pragma unroll
  for (int j = 0; j < V; ++j) {
    u32x4* row = lds + (V * cg + j) * GR;  // destination row V cg + j
#pragma unroll
    for (int h = 0; h < H; ++h)
      row[(rg * H + h) ^ (cg & (GR - 1))] =
          kEs == 2 ? column8(a, j) : u32x4{a[(4 * h) & 7][j & 3], a[(4 * h + 1) & 7][j & 3], a[(4 * h + 2) & 7][j & 3], a[(4 * h + 3) & 7][j & 3]};
  }
  __syncthreads();
  const int w = threadIdx.x % GR, r0 = threadIdx.x / GR;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int row = r0 + (kTileThreads / GR) * k;
    u32x4* p = reinterpret_cast<u32x4*>(dst + (uint64_t(row) * t.dst_ld + V * w) * kEs);
    if (kNt)
      st(lds[row * GR + (w ^ ((row / V) & (GR - 1)))], p);
    else
      *p = lds[row * GR + (w ^ ((row / V) & (GR - 1)))];
  }
}

template <bool kPlain>
__global__ __launch_bounds__(kTileThreads) void wb_tile_kernel(const Task* __restrict__ tasks,
                                                               const uint64_t* __restrict__ ptrs, const char* buf,
                                                               const char* aux) {
  __shared__ u32x4 lds[kTileRows * kTileCols / 8];
  const Task t = tasks[blockIdx.x];
  const char* src = base_of(t.src_idx, ptrs, buf, aux) + t.src_off;
  char* dst = const_cast<char*>(base_of(t.dst_idx, ptrs, buf, aux)) + t.dst_off;
  if (t.sdt == WB_F32)
    run_tile<4, !kPlain>(t, src, dst, lds);
  else
    run_tile<2, true>(t, src, dst, lds);
}

// ---- fp8 E4M3FN blocks ---------------------------------------------------

namespace {

__device__ __forceinline__ float load_f32(const char* p, int dt) {
  return dt == WB_F32 ? *reinterpret_cast<const float*>(p) : __uint_as_float(uint32_t(*reinterpret_cast<const uint16_t*>(p)) << 16);
}

// Address of element (r, c) of the block in its pieces of es-byte elements.
__device__ __forceinline__ const char* find_one(const QPiece* pcs, uint32_t n, const char* recv, int r, int c, int es) {
  for (uint32_t i = 0; i < n; ++i) {
    const QPiece& p = pcs[i];
    if (r >= p.r0 && r <= p.r1m1 && c >= p.c0 && c <= p.c1m1)
      return recv + p.src_off + (uint64_t(r - p.r0) * p.src_ld + (c - p.c0)) * es;
  }
  return nullptr;
}

// Element (r, c) of the block from its pieces (the block is exactly covered).
__device__ __forceinline__ float gather_one(const QPiece* pcs, int n, const char* recv, int r, int c) {
  for (int i = 0; i < n; ++i) {
    const QPiece& p = pcs[i];
    if (r >= p.r0 && r <= p.r1m1 && c >= p.c0 && c <= p.c1m1) {
      const int es = p.sdt == WB_F32 ? 4 : 2;
      return load_f32(recv + p.src_off + (uint64_t(r - p.r0) * p.src_ld + (c - p.c0)) * es, p.sdt);
    }
  }
  return 0.0f;
}

__device__ __forceinline__ void unpack8(const u32x4 x, float* v) {
  v[0] = bf16_lo(x.x); v[1] = bf16_hi(x.x); v[2] = bf16_lo(x.y); v[3] = bf16_hi(x.y);
  v[4] = bf16_lo(x.z); v[5] = bf16_hi(x.z); v[6] = bf16_lo(x.w); v[7] = bf16_hi(x.w);
}

constexpr int kLdsPieces = 128;

// The block's scale s = amax / 448 (IEEE division; 1 for an all-zero block)
// and the quantities RN(x / s) is computed from, s = m 2^E (m in [1, 2)):
//
// mode 2 (bf16 source, -90 <= E <= 100): r = RN(1 / s), q0 = RN(x r),
//   e = x - q0 s (exact, by FMA), q = RN(q0 + e r). A quotient that can round
//   to a non-zero E4M3 value has |x / s| >= 2^-10, so q0 >= 2^-10, e is at
//   least 2^(E - 33) in magnitude and every intermediate is a normal number;
//   r stays normal for E <= 100.
// mode 1 (bf16 source, any other normal s): the same on x' = x 2^-E and m,
//   which keeps the intermediates normal whatever E.
// In both the sign is copied from x: a quotient that rounds to zero can lose
//   it in the correction. Since |x| <= amax, |q| <= 448.00003 rounds to at most
//   448 in E4M3, so no clamp is needed. Both are verified exhaustively for
//   every bf16 (x, amax) pair.
// mode 3 (fp32 source, -90 <= E <= 100, m not all ones): the same with a
//   second correction: q0 = RN(x r) is within 2 ulp, q1 = RN(q0 + e0 r) then
//   within 1, and for such a q1, r = RN(1 / s) and e1 = x - q1 s (exact)
//   RN(q1 + e1 r) is RN(x / s) (Markstein's theorem, which excludes an s whose
//   significand is all ones). Where |x / s| < 2^-11 the steps may underflow;
//   the result then still rounds to zero. 6 operations instead of the about
//   12 of a division. Clamped like mode 0, so a NaN gives what it gave there.
// mode 0 (other fp32 sources, subnormal s): IEEE division, clamped to +-448 (a
//   no-op that keeps the conversion away from its overflow path whatever the
//   source).
struct QScale {
  float s, sp, rp, pw;
  int mode;
};

__device__ __forceinline__ QScale make_scale(float amax, bool bf16_source) {
  QScale q;
  q.s = amax > 0.0f ? amax / 448.0f : 1.0f;  // IEEE fp32 division
  const uint32_t sbits = __float_as_uint(q.s);
  const int sexp = int((sbits >> 23) & 0xFF);  // E + 127
  const bool mid = sexp >= 127 - 90 && sexp <= 127 + 100;
  q.mode = sexp == 0 ? 0 : bf16_source ? (mid ? 2 : 1) : (mid && (sbits & 0x007FFFFFu) != 0x007FFFFFu) ? 3 : 0;
  q.pw = __uint_as_float(uint32_t(254 - sexp) << 23);  // 2^-E
  q.sp = q.mode == 1 ? __uint_as_float((sbits & 0x007FFFFFu) | 0x3F800000u) : q.s;  // m, or s
  q.rp = 1.0f / q.sp;
  return q;
}

template <int kMode>
__device__ __forceinline__ float quotient(float x, const QScale& q) {
  if (kMode == 0) return __builtin_amdgcn_fmed3f(x / q.s, -448.0f, 448.0f);
  if (kMode == 3) {
    const float q0 = x * q.rp;
    const float q1 = fmaf(fmaf(-q0, q.s, x), q.rp, q0);
    const float q2 = fmaf(fmaf(-q1, q.s, x), q.rp, q1);
    return __builtin_amdgcn_fmed3f(__builtin_copysignf(q2, x), -448.0f, 448.0f);
  }
  const float xp = kMode == 1 ? x * q.pw : x;
  const float q0 = xp * q.rp;
  const float e = fmaf(-q0, q.sp, xp);
  return __builtin_copysignf(fmaf(e, q.rp, q0), x);
}

// E4M3FN(RN(x / s)) of this thread's R rows of 8 columns (rows rb + kStep k),
// row k's values produced by row(k, v); 8-byte stores, or bytes at a ragged
// right edge or an unaligned destination.
template <int kMode, int R, int kStep, class Row>
__device__ __forceinline__ void quantise_store(Row row, const QScale& qs, int rows, int cols, int rb, int cg,
                                               uint8_t* q8, uint32_t dst_ld, bool vec) {
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = rb + kStep * k;
    if (r >= rows || cg >= cols) continue;
    float v[8], q[8];
    row(k, v);
#pragma unroll
    for (int m = 0; m < 8; ++m) q[m] = quotient<kMode>(v[m], qs);
    uint32_t lo = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], lo, true);
    uint32_t hi = __builtin_amdgcn_cvt_pk_fp8_f32(q[4], q[5], 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(q[6], q[7], hi, true);
    uint8_t* dst = q8 + uint64_t(r) * dst_ld + cg;
    if (vec && cg + 8 <= cols) {
      st(u32x2{lo, hi}, reinterpret_cast<u32x2*>(dst));
    } else {
#pragma unroll
      for (int m = 0; m < 8; ++m)
        if (cg + m < cols) dst[m] = static_cast<uint8_t>((m < 4 ? lo : hi) >> (8 * (m & 3)));
    }
  }
}

template <int R, int kStep, class Row>
__device__ __forceinline__ void quantise_block(Row row, const QScale& qs, int rows, int cols, int rb, int cg,
                                               uint8_t* q8, uint32_t dst_ld, bool vec) {
  // the mode is uniform over the block, so this branch is taken once, outside
  // the element loops
  if (qs.mode == 2)
    quantise_store<2, R, kStep>(row, qs, rows, cols, rb, cg, q8, dst_ld, vec);
  else if (qs.mode == 1)
    quantise_store<1, R, kStep>(row, qs, rows, cols, rb, cg, q8, dst_ld, vec);
  else
    quantise_store<0, R, kStep>(row, qs, rows, cols, rb, cg, q8, dst_ld, vec);
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Takes the word by value: __builtin_bit_cast applied to a vector element
// expression (v.y) reads the vector's first element in this compiler.
__device__ __forceinline__ u16x2 as_u16x2(uint32_t w) { return __builtin_bit_cast(u16x2, w); }

// Per-lane view of one of the two blocks of a pair.
struct PairLane {
  const char* src;   // this lane's first element (row rb, column cg)
  uint64_t src_ld2;  // wire row stride in bytes
  uint8_t* q8;       // fp8 block origin
  uint32_t dst_ld;
  int rows, cols;
  bool vec;
};

// Blocks i0 and i0 + 1 (absent when i0 + 1 == nsingle), both pairable. In
// each half-wave, lanes 0..15 take block i0 and lanes 16..31 block i0 + 1, so a
// load instruction reads 512 contiguous bytes of each of two rows when the two
// blocks are neighbours on the wire; thread t holds columns 8 (t mod 16) .. + 7
// of rows t / 32 + 8 k, k < 16, as raw bf16. kFull: both blocks present,
// 128 x 128 and with 8-byte stores, so no load or store needs a predicate.
// kBands: at least one block of the pair is QB_BANDS; each row's source is
// base + r * ld2 of the band that holds it, from the lane's own block's band
// table (registers: indexed only by unrolled constants); otherwise every row
// follows the single piece's stride.
struct PairBands {
  uint64_t base[kMaxBands];   // recv + band offset - first row * pitch (bytes)
  uint32_t ld2[kMaxBands];    // band pitch in bytes
  uint32_t start[kMaxBands];  // first row; bands past the block's last: 256
};

template <bool kFull, bool kBands>
__device__ __forceinline__ void qblock_pair_run(const PairLane& L, const PairBands& S, int h, bool on,
                                                const QBlock& b0, const QBlock& b1, const uint64_t* __restrict__ ptrs) {
  constexpr int R = 16, kStep = 8;
  static_assert(kQBlockThreads == 32 * kStep, "pair mapping");
  static_assert(kMaxBands == 4, "band selection");
  __shared__ uint32_t wave_max[kQBlockThreads / 64][2];
  const int cg = (threadIdx.x & 15) * 8, rb = threadIdx.x >> 5;
  u32x4 raw[R];
  if (kBands) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t r = rb + kStep * k;
      raw[k] = u32x4{0u, 0u, 0u, 0u};
      if (kFull || (int(r) < L.rows && cg < L.cols)) {
        uint64_t base = S.base[0];
        uint32_t ld2 = S.ld2[0];
#pragma unroll
        for (int j = 1; j < kMaxBands; ++j)
          if (r >= S.start[j]) {
            base = S.base[j];
            ld2 = S.ld2[j];
          }
        raw[k] = ld(reinterpret_cast<const u32x4*>(global_ptr(base + uint64_t(r) * ld2 + uint64_t(cg) * 2)));
      }
    }
  } else if (kFull) {
    const char* p = L.src;
#pragma unroll
    for (int k = 0; k < R; ++k, p += kStep * L.src_ld2) raw[k] = ld(reinterpret_cast<const u32x4*>(p));
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int r = rb + kStep * k;
      raw[k] = u32x4{0u, 0u, 0u, 0u};
      if (r < L.rows && cg < L.cols)
        raw[k] = ld(reinterpret_cast<const u32x4*>(L.src + uint64_t(kStep * k) * L.src_ld2));
    }
  }
  // amax: finite bf16 magnitudes order as their bit patterns with the sign
  // cleared (two per word, packed 16-bit maxima)
  u16x2 acc = {0, 0};
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const u32x4 a = raw[k] & 0x7FFF7FFFu;
    acc = __builtin_elementwise_max(acc, as_u16x2(a.x));
    acc = __builtin_elementwise_max(acc, as_u16x2(a.y));
    acc = __builtin_elementwise_max(acc, as_u16x2(a.z));
    acc = __builtin_elementwise_max(acc, as_u16x2(a.w));
  }
  uint32_t m = max(uint32_t(acc.x), uint32_t(acc.y));
  // lanes of one block: xor 1..8 within a 16-lane group, xor 32 across the
  // half-waves
  m = max(m, uint32_t(__shfl_xor(int(m), 1)));
  m = max(m, uint32_t(__shfl_xor(int(m), 2)));
  m = max(m, uint32_t(__shfl_xor(int(m), 4)));
  m = max(m, uint32_t(__shfl_xor(int(m), 8)));
  m = max(m, uint32_t(__shfl_xor(int(m), 32)));
  if ((threadIdx.x & 47) == 0) wave_max[threadIdx.x >> 6][h] = m;  // lanes 0 and 16
  __syncthreads();
  m = wave_max[0][h];
#pragma unroll
  for (int w = 1; w < kQBlockThreads / 64; ++w) m = max(m, wave_max[w][h]);
  const QScale qs = make_scale(__uint_as_float(m << 16), true);
  // rows and columns past the edge are skipped by the store loop; in the full
  // case there are none
  const int rows = kFull ? 128 : L.rows, cols = kFull ? 128 : L.cols;
  quantise_block<R, kStep>([&](int k, float* v) { unpack8(raw[k], v); }, qs, rows, cols, rb, cg, L.q8, L.dst_ld,
                           kFull || L.vec);
  const QBlock& b = h ? b1 : b0;
  if (on && (threadIdx.x & ~16u) == 0) reinterpret_cast<float*>(global_ptr(ptrs[b.scale_idx]))[b.scale_off] = qs.s;
}

// This lane's view of the block it works on in a pair (h: 0 or 1).
__device__ __forceinline__ PairLane pair_lane(const QBlock& b0, const QBlock& b1, int h, bool on,
                                              const uint64_t* __restrict__ ptrs, const char* recv) {
  const QBlock& b = h ? b1 : b0;
  const int cg = (threadIdx.x & 15) * 8, rb = threadIdx.x >> 5;
  PairLane L;
  L.src_ld2 = uint64_t(b.src_ld) * 2;
  L.src = recv + b.src_off + uint64_t(cg) * 2 + uint64_t(rb) * L.src_ld2;
  L.dst_ld = b.dst_ld;
  uint8_t* const q0 = reinterpret_cast<uint8_t*>(global_ptr(ptrs[b0.dst_idx])) + b0.dst_off;
  uint8_t* const q1 = reinterpret_cast<uint8_t*>(global_ptr(ptrs[b1.dst_idx])) + b1.dst_off;
  L.q8 = h ? q1 : q0;
  L.rows = on ? b.rows_m1 + 1 : 0;
  L.cols = b.cols_m1 + 1;
  L.vec = (b.flags & QB_VEC_STORE) != 0;
  return L;
}

// Blocks i0 and i0 + 1, both QB_SINGLE, 128 x 128, 8-byte stores (the
// planner's full pairs): no predicates, one quotient form per block.
__device__ __forceinline__ void qblock_pair_full(const QBlock* __restrict__ blocks, uint32_t i0, const uint64_t* __restrict__ ptrs,
                                 const char* recv) {
  const QBlock b0 = blocks[i0];
  const QBlock b1 = blocks[i0 + 1];
  const int h = (threadIdx.x >> 4) & 1;
  qblock_pair_run<true, false>(pair_lane(b0, b1, h, true, ptrs, recv), PairBands{}, h, true, b0, b1, ptrs);
}

// Blocks i0 and i0 + 1 (absent when i0 + 1 == n), both pairable, any extent.
__device__ __forceinline__ void qblock_pair(const QBlock* __restrict__ blocks, uint32_t i0, uint32_t n,
                            const QPiece* __restrict__ pieces, const uint64_t* __restrict__ ptrs, const char* recv) {
  // both descriptors are read at workgroup-uniform addresses; each lane then
  // selects its block's fields
  const bool has1 = i0 + 1 < n;
  const QBlock b0 = blocks[i0];
  const QBlock b1 = blocks[has1 ? i0 + 1 : i0];
  const int h = (threadIdx.x >> 4) & 1;
  const bool on = h == 0 || has1;
  const PairLane L = pair_lane(b0, b1, h, on, ptrs, recv);
  const bool full = has1 && b0.rows_m1 == 127 && b0.cols_m1 == 127 && b1.rows_m1 == 127 && b1.cols_m1 == 127 &&
                    (b0.flags & b1.flags & QB_VEC_STORE);
  const bool bands = ((b0.flags | b1.flags) & QB_BANDS) != 0;  // uniform over the workgroup
  if (bands) {
    // the band table of this lane's block (its own stride when it is a
    // single piece)
    const uint32_t flags = h ? b1.flags : b0.flags;
    const uint32_t np = h ? b1.npieces : b0.npieces, p0 = h ? b1.piece0 : b0.piece0;
    PairBands S;
#pragma unroll
    for (int j = 0; j < kMaxBands; ++j) {
      S.base[j] = 0;
      S.ld2[j] = 0;
      S.start[j] = 256;
    }
    if (flags & QB_BANDS) {
#pragma unroll
      for (int j = 0; j < kMaxBands; ++j)
        if (uint32_t(j) < np) {
          const QPiece q = pieces[p0 + j];
          S.ld2[j] = q.src_ld * 2;
          S.base[j] = reinterpret_cast<uint64_t>(recv) + q.src_off - uint64_t(q.r0) * S.ld2[j];
          S.start[j] = q.r0;
        }
    } else {
      S.ld2[0] = (h ? b1.src_ld : b0.src_ld) * 2;
      S.base[0] = reinterpret_cast<uint64_t>(recv) + (h ? b1.src_off : b0.src_off);
      S.start[0] = 0;
    }
    if (full)
      qblock_pair_run<true, true>(L, S, h, on, b0, b1, ptrs);
    else
      qblock_pair_run<false, true>(L, S, h, on, b0, b1, ptrs);
  } else if (full) {
    qblock_pair_run<true, false>(L, PairBands{}, h, on, b0, b1, ptrs);
  } else {
    qblock_pair_run<false, false>(L, PairBands{}, h, on, b0, b1, ptrs);
  }
}

// Where the 16-byte chunks of the block's rows come from: a block that is
// one wire piece (QB_DIRECT) keeps its address in the descriptor; otherwise
// the piece list is staged in LDS with a row -> piece table for the pieces
// that span the block's full width (row bands: a replicated tensor split by
// rows among its senders, a flat shard cut between rows). Rows with none
// search the list.
enum SourceKind { kSourceDirect, kSourceStaged, kSourceList };
template <int kKind>
struct BlockSource {
  const char* base;          // direct: the block's first element
  const QPiece* pcs;         // staged: in LDS; list: in memory
  const uint8_t* row_piece;  // staged
  uint32_t ld, n;
  template <bool kF32>
  __device__ __forceinline__ const char* at(const char* recv, int r, int c) const {
    constexpr int es = kF32 ? 4 : 2, V = 16 / es;
    if (kKind == kSourceDirect) return base + (uint64_t(r) * ld + c) * es;
    uint32_t i = kKind == kSourceStaged ? row_piece[r] : 0xFF;
    if (i == 0xFF)
      for (i = 0; i < n; ++i) {
        const QPiece& p = pcs[i];
        if (r >= p.r0 && r <= p.r1m1 && c >= p.c0 && c + V - 1 <= p.c1m1) break;
      }
    if (i >= n) return nullptr;  // the chunk straddles pieces
    const QPiece& p = pcs[i];
    return recv + p.src_off + (uint64_t(r - p.r0) * p.src_ld + (c - p.c0)) * es;
  }
  template <bool kF32>
  __device__ __forceinline__ const char* one(const char* recv, int r, int c) const {
    constexpr int es = kF32 ? 4 : 2;
    if (kKind == kSourceDirect) return base + (uint64_t(r) * ld + c) * es;
    return find_one(pcs, n, recv, r, c, es);
  }
};

// One block of any kind: a thread holds 16-byte chunks of V wire elements (8
// bf16 or 4 fp32) of up to R rows, T threads a row (fewer for blocks of at
// most half or a quarter of 128 columns). A row of 128 is 256 (512) contiguous
// bytes of a load instruction; sources may sit at any element address and the
// fp8 rows at any byte. The last chunk of a row whose width is no multiple of
// V is moved left over its neighbour (the same values, written twice).
// Bound: HBM; 8 (16) 16-byte loads per thread are in flight at once. An fp32
// rank of half an 8 B dense model (7.0 GB of blocks in, 1.7 GB out): 8.22 ms when
// every element searched its piece, 1.46 ms now (6.0 TB/s). For bf16, chunks of
// 4 elements on 32 threads a row made blocks of 32 row bands 6 % slower than
// 8 on 16: twice the row lookups.
template <bool kF32, int kKind>
__device__ __forceinline__ void qblock_wide(const QBlock& b, const BlockSource<kKind>& S, const uint64_t* __restrict__ ptrs,
                                            const char* recv) {
  constexpr int es = kF32 ? 4 : 2, V = 16 / es, T0 = kF32 ? 5 : 4, R = 128 >> (8 - T0);
  static_assert(kQBlockThreads == 256 && (V << T0) == 128 && (R << (8 - T0)) == 128, "block mapping");
  __shared__ float wave_max[kQBlockThreads / 64];
  const int rows = b.rows_m1 + 1, cols = b.cols_m1 + 1;
  const int sh = cols > 64 ? T0 : cols > 32 ? T0 - 1 : T0 - 2;  // log2 T
  const int step = kQBlockThreads >> sh, rb = threadIdx.x >> sh;
  const int c0 = int(threadIdx.x & ((1u << sh) - 1u)) * V;
  const bool on = c0 < cols;
  const int cg = min(c0, max(cols - V, 0));
  const bool whole = cols >= V;
  u32x4 raw[R];
  bool odd = false;  // some chunk of this lane needs single elements
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = rb + step * k;
    raw[k] = u32x4{0u, 0u, 0u, 0u};
    if (!on || r >= rows) continue;
    const char* p = whole ? S.template at<kF32>(recv, r, cg) : nullptr;
    if (p)
      raw[k] = ld_at<u32x4, 2>(p);
    else
      odd = true;
  }
  if (odd) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int r = rb + step * k;
      if (r >= rows || (whole && S.template at<kF32>(recv, r, cg))) continue;
      uint32_t e[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int m = 0; m < V; ++m) {
        if (cg + m >= cols) break;
        const char* p = S.template one<kF32>(recv, r, cg + m);
        if (!p) continue;
        if (kF32)
          e[m & 3] = *reinterpret_cast<const uint32_t*>(p);
        else
          e[m >> 1] |= uint32_t(*reinterpret_cast<const uint16_t*>(p)) << (16 * (m & 1));
      }
      raw[k] = u32x4{e[0], e[1], e[2], e[3]};
    }
  }
  auto values = [&](int k, float* v) {
    if (kF32) {
#pragma unroll
      for (int m = 0; m < 4; ++m) v[m] = __uint_as_float(raw[k][m]);
    } else {
      unpack8(raw[k], v);
    }
  };
  float amax = 0.0f;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    float v[V];
    values(k, v);
#pragma unroll
    for (int m = 0; m < V; ++m) amax = fmaxf(amax, fabsf(v[m]));
  }
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = amax;
  __syncthreads();
  amax = wave_max[0];
#pragma unroll
  for (int w = 1; w < kQBlockThreads / 64; ++w) amax = fmaxf(amax, wave_max[w]);
  const QScale qs = make_scale(amax, !kF32);
  if (threadIdx.x == 0) reinterpret_cast<float*>(global_ptr(ptrs[b.scale_idx]))[b.scale_off] = qs.s;
  if (!on) return;
  uint8_t* q8 = reinterpret_cast<uint8_t*>(global_ptr(ptrs[b.dst_idx])) + b.dst_off + cg;
  auto store = [&](auto mode) {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int r = rb + step * k;
      if (r >= rows) continue;
      float v[V], q[V];
      values(k, v);
#pragma unroll
      for (int m = 0; m < V; ++m) q[m] = quotient<mode.value>(v[m], qs);
      uint32_t w[V / 4];
#pragma unroll
      for (int m = 0; m < V / 4; ++m) {
        w[m] = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * m], q[4 * m + 1], 0, false);
        w[m] = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * m + 2], q[4 * m + 3], w[m], true);
      }
      uint8_t* dst = q8 + uint64_t(r) * b.dst_ld;
      if (!whole) {
#pragma unroll
        for (int m = 0; m < V; ++m)
          if (m < cols) dst[m] = static_cast<uint8_t>(w[m / 4] >> (8 * (m & 3)));
      } else if (kF32) {
        st_at<uint32_t, 1>(w[0], dst);
      } else {
        st_at<u32x2, 1>(u32x2{w[0], w[V / 4 - 1]}, dst);
      }
    }
  };
  // the mode is uniform over the block
  if (kF32) {
    if (qs.mode == 3)
      store(std::integral_constant<int, 3>{});
    else
      store(std::integral_constant<int, 0>{});
  } else if (qs.mode == 2) {
    store(std::integral_constant<int, 2>{});
  } else if (qs.mode == 1) {
    store(std::integral_constant<int, 1>{});
  } else {
    store(std::integral_constant<int, 0>{});
  }
}

// A block whose pieces are neither all bf16 nor all fp32: 8 rows of 8 columns
// per thread, held as fp32. A row's chunk of 8 that lies in one piece is one
// (bf16) or two (fp32) loads of 16 bytes, all in flight together; the others are
// searched for element by element. 8192 x 8192 in bands of 64 rows of both types
// took 343 us when every element was searched for and 66 now, in strips of 64
// columns 521 and 84.
template <bool kStaged>
__device__ __forceinline__ void qblock_mixed(const QBlock& b, const QPiece* pcs, const uint8_t* row_piece,
                                             const uint64_t* __restrict__ ptrs, const char* recv) {
  constexpr int R = 8, kStep = 16;
  static_assert(kQBlockThreads == 16 * kStep, "block mapping");
  __shared__ float wave_max[kQBlockThreads / 64];
  const int rows = b.rows_m1 + 1, cols = b.cols_m1 + 1;
  const int cg = (threadIdx.x & 15) * 8, rb = threadIdx.x >> 4;
  const uint32_t n = b.npieces;
  u32x4 lo[R], hi[R];
  unsigned wide = 0, odd = 0;  // bit k: row k's chunk is fp32; needs single elements
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = rb + kStep * k;
    lo[k] = hi[k] = u32x4{0u, 0u, 0u, 0u};
    if (r >= rows || cg >= cols) continue;
    uint32_t i = kStaged ? row_piece[r] : 0xFF;
    if (i == 0xFF || cg + 7 >= cols)
      for (i = 0; i < n; ++i) {
        const QPiece& p = pcs[i];
        if (r >= p.r0 && r <= p.r1m1 && cg >= p.c0 && cg + 7 <= p.c1m1) break;
      }
    if (i >= n) {
      odd |= 1u << k;
      continue;
    }
    const QPiece& p = pcs[i];
    const int es = p.sdt == WB_F32 ? 4 : 2;
    const char* a = recv + p.src_off + (uint64_t(r - p.r0) * p.src_ld + (cg - p.c0)) * es;
    lo[k] = ld_at<u32x4, 2>(a);
    if (es == 4) {
      wide |= 1u << k;
      hi[k] = ld_at<u32x4, 2>(a + 16);
    }
  }
  float v[R][8], amax = 0.0f;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = rb + kStep * k;
    unpack8(lo[k], v[k]);
    if ((wide >> k) & 1u) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        v[k][m] = __uint_as_float(lo[k][m]);
        v[k][4 + m] = __uint_as_float(hi[k][m]);
      }
    }
    if ((odd >> k) & 1u) {
#pragma unroll
      for (int m = 0; m < 8; ++m) v[k][m] = cg + m < cols ? gather_one(pcs, n, recv, r, cg + m) : 0.0f;
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) amax = fmaxf(amax, fabsf(v[k][m]));
  }
  for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = amax;
  __syncthreads();
  amax = wave_max[0];
#pragma unroll
  for (int w = 1; w < kQBlockThreads / 64; ++w) amax = fmaxf(amax, wave_max[w]);
  const QScale qs = make_scale(amax, true);
  QScale q0 = qs;
  q0.mode = 0;
  uint8_t* q8 = reinterpret_cast<uint8_t*>(global_ptr(ptrs[b.dst_idx])) + b.dst_off;
  quantise_store<0, R, kStep>(
      [&](int k, float* out) {
#pragma unroll
        for (int m = 0; m < 8; ++m) out[m] = v[k][m];
      },
      q0, rows, cols, rb, cg, q8, b.dst_ld, (b.flags & QB_VEC_STORE) != 0);
  if (threadIdx.x == 0) reinterpret_cast<float*>(global_ptr(ptrs[b.scale_idx]))[b.scale_off] = qs.s;
}

__device__ __forceinline__ void qblock_one(const QBlock& b, const QPiece* __restrict__ pieces, const uint64_t* __restrict__ ptrs,
                           const char* recv) {
  __shared__ QPiece lds_pcs[kLdsPieces];
  __shared__ uint8_t row_piece[128];
  const bool mixed = !(b.flags & (QB_BF16_SOURCE | QB_F32_SOURCE));
  const bool f32 = (b.flags & QB_F32_SOURCE) != 0;
  const uint32_t n = b.npieces;
  if (b.flags & QB_DIRECT) {
    const BlockSource<kSourceDirect> S{recv + b.src_off, nullptr, nullptr, b.src_ld, 0u};
    if (f32)
      qblock_wide<true>(b, S, ptrs, recv);
    else
      qblock_wide<false>(b, S, ptrs, recv);
  } else if (n <= kLdsPieces) {  // at least one piece
    for (uint32_t i = threadIdx.x; i < n; i += kQBlockThreads) lds_pcs[i] = pieces[b.piece0 + i];
    if (threadIdx.x < 128) row_piece[threadIdx.x] = 0xFF;
    __syncthreads();
    // 256 / n threads per piece mark its rows
    const uint32_t i = threadIdx.x % n, part = threadIdx.x / n, parts = kQBlockThreads / n;
    const QPiece& p = lds_pcs[i];
    if (part < parts && p.c0 == 0 && p.c1m1 == b.cols_m1)
      for (uint32_t r = p.r0 + part; r <= p.r1m1; r += parts) row_piece[r] = static_cast<uint8_t>(i);
    __syncthreads();
    const BlockSource<kSourceStaged> S{nullptr, lds_pcs, row_piece, 0u, n};
    if (mixed)
      qblock_mixed<true>(b, lds_pcs, row_piece, ptrs, recv);
    else if (f32)
      qblock_wide<true>(b, S, ptrs, recv);
    else
      qblock_wide<false>(b, S, ptrs, recv);
  } else {
    const BlockSource<kSourceList> S{nullptr, pieces + b.piece0, nullptr, 0u, n};
    if (mixed)
      qblock_mixed<false>(b, pieces + b.piece0, nullptr, ptrs, recv);
    else if (f32)
      qblock_wide<true>(b, S, ptrs, recv);
    else
      qblock_wide<false>(b, S, ptrs, recv);
  }
}

}  // namespace

// The fp8 blocks of a launch range come in three classes, taken by one launch
// (the slower classes overlap the bulk instead of trailing it in launches of
// their own): workgroup w < nfull / 2 takes the full pair 2v, 2v + 1, v = w in
// XCD-aware order; the next
// ones the other pairable blocks two at a time (the second absent past npair);
// the rest one block each.
__global__ __launch_bounds__(kQBlockThreads) void wb_qblock_kernel(const QBlock* __restrict__ blocks,
                                                                   const QPiece* __restrict__ pieces,
                                                                   const uint64_t* __restrict__ ptrs,
                                                                   const char* recv, uint32_t n, uint32_t nfull,
                                                                   uint32_t npair) {
  const uint32_t g0 = nfull / 2, g1 = (npair - nfull + 1) / 2;
  if (blockIdx.x < g0) {
    qblock_pair_full(blocks, 2 * uint32_t(xcd_order(blockIdx.x, g0, kXcdRunPairs)), ptrs, recv);
  } else if (blockIdx.x < g0 + g1) {
    qblock_pair(blocks + nfull, 2 * (blockIdx.x - g0), npair - nfull, pieces, ptrs, recv);
  } else {
    // in XCD-aware order too: blocks of one wire row band are neighbours
    const uint32_t i = npair + uint32_t(xcd_order(blockIdx.x - g0 - g1, n - npair, kXcdRunPairs));
    if (i < n) qblock_one(blocks[i], pieces, ptrs, recv);
  }
}

void task_grid(uint32_t n, const TaskSplit& sp, uint32_t* gx, uint32_t* gy) {
  const uint64_t total =
      (uint64_t(sp.n[0]) << sp.s[0]) + (uint64_t(sp.n[1]) << sp.s[1]) + (n - sp.n[0] - sp.n[1] - sp.tiles);
  if (total == 0) {
    *gx = *gy = 0;
    return;
  }
  if (total <= kMaxGridX) {
    *gx = static_cast<uint32_t>(total);
    *gy = 1;
  } else {  // fewest rows, then the narrowest rows: fewer than gy idle workgroups
    *gy = static_cast<uint32_t>((total + kMaxGridX - 1) / kMaxGridX);
    *gx = static_cast<uint32_t>((total + *gy - 1) / *gy);
  }
}

int launch_tasks(const Task* tasks, uint32_t n, const TaskSplit& sp, const uint64_t* ptrs, const void* buf,
                 const void* aux, void* stream) {
  if (n == 0) return hipSuccess;
  uint32_t gx, gy;
  task_grid(n, sp, &gx, &gy);
  if (gx) {
    hipLaunchKernelGGL(wb_tasks_kernel, dim3(gx, gy), dim3(kThreads), WB_TASK_DYN_LDS,
                       static_cast<hipStream_t>(stream), tasks, ptrs, static_cast<const char*>(buf),
                       static_cast<const char*>(aux), n - sp.tiles, sp.n[0], sp.n[1], sp.s[0], sp.s[1]);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (sp.tiles) {
    const auto kernel = sp.tiles <= kPlainTiles ? wb_tile_kernel<true> : wb_tile_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(sp.tiles), dim3(kTileThreads), 0, static_cast<hipStream_t>(stream),
                       tasks + (n - sp.tiles), ptrs, static_cast<const char*>(buf), static_cast<const char*>(aux));
    return hipGetLastError();
  }
  return hipSuccess;
}

int launch_qblocks(const QBlock* blocks, uint32_t n, uint32_t nfull, uint32_t npair, const QPiece* pieces,
                   const uint64_t* ptrs, const void* buf, void* stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(wb_qblock_kernel, dim3(qblock_workgroups(n, nfull, npair)), dim3(kQBlockThreads),
                     n - npair > npair ? kQBlockLdsSingles : kQBlockLdsPairs, static_cast<hipStream_t>(stream), blocks,
                     pieces, ptrs, static_cast<const char*>(buf), n, nfull, npair);
  return hipGetLastError();
}

const char* hip_error_string(int err) { return hipGetErrorString(static_cast<hipError_t>(err)); }

}  // namespace wb
