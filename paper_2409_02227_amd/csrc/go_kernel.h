// go_kernel.h -- what every GO-Kernel shares: types, MFMA wrappers, buffer
// access, tile order, element-wise add members and the split-K reduction.
//
// GOLDYLOC (Sec. 2.1.3 and Sec. 4.2) treats a GEMM kernel as a tiled loop:
// each workgroup owns one C tile and walks K, staging operand tiles in LDS;
// tile size, workgroup count, occupancy and memory traffic are the features
// that decide how well kernels share the GPU when several run at once.  The
// GO-Kernels (go_kernel_p.h: 256 x 256 tiles; go_kernel_u.h: every smaller one)
// expose those knobs as template parameters (macro tile, waves per workgroup,
// stages) and launch parameters (grid cap, tile order), so the offline tuner
// can pick one per GEMM shape and concurrency degree.
//
// Results: acc * scale (fp8 per-tensor scales, 1 otherwise), rounded to
// nearest-even into bf16 (bf16 and fp8 inputs) or fp16 (fp16 inputs), fp32 as
// is.  beta = 0: C is overwritten.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gdy_internal.h"

namespace gdy {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

template <int DT> struct ElemSize;
template <> struct ElemSize<DT_BF16> { static constexpr int v = 2; };
template <> struct ElemSize<DT_F16> { static constexpr int v = 2; };
template <> struct ElemSize<DT_FP8> { static constexpr int v = 1; };
template <> struct ElemSize<DT_F32> { static constexpr int v = 4; };

// Bytes of one output element: fp32 inputs give fp32 results, the others
// round to a 16-bit type.
template <int DT> struct OutSize { static constexpr int v = 2; };
template <> struct OutSize<DT_F32> { static constexpr int v = 4; };

// ---------------------------------------------------------------------------
// MFMA wrappers.  An operand is one lane's fragment (lds_copy.h: FragT); Acc is
// one lane's share of a 16 x 16 block.
// Output layout (CDNA matrix-core convention): accumulator r of lane l is row
// 4*(l/16) + r, column l%16.  Lanes l and l' with l%16 equal hold the same row
// of A (column of B) at different K offsets; A and B use the same K
// assignment, so any consistent lane->K mapping is a valid sum.
// ---------------------------------------------------------------------------
template <int DT, int MM> struct Mma;

template <> struct Mma<DT_BF16, 16> {
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<DT_F16, 16> {
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
// fp8: the f8f6f4 MFMAs with format 0 (OCP E4M3) for both operands and unit
// block scales (E8M0 exponent 127 = 2^0).  32 bytes of K per lane.
template <> struct Mma<DT_FP8, 16> {
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  static __device__ __forceinline__ Acc run(i32x8 a, i32x8 b, Acc c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
  }
};

// fp32: one element of K per lane.
template <> struct Mma<DT_F32, 16> {
  typedef f32x4 Acc;
  static constexpr int NACC = 4;
  static __device__ __forceinline__ Acc run(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Global reads and writes go through raw buffer resources with 32-bit byte
// offsets.  The buffer size is the operand's extent rounded up to the end of the
// dword holding its last byte (the unit range-checks whole dwords, and that
// dword is always mapped): a read beyond it returns zero and never touches
// memory.
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr int kRsrcWord3 = 0x00020000;  // raw 32-bit data format, gfx9 family

__device__ __forceinline__ Rsrc make_rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, kRsrcWord3);
}

template <int ES>
__device__ __forceinline__ unsigned load_elem(Rsrc r, int off) {
  if (ES == 4) return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  if (ES == 2) return (unsigned)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
  return (unsigned)__builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
}

// fp32 -> output elements, round to nearest even, by the conversion
// instructions (two elements each; rounding by integer arithmetic took six
// operations an element, 3 us of a 256 x 256 tile's epilogue).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
template <int DT> __device__ __forceinline__ unsigned to_out2(float lo, float hi) {
  const f32x2 x = {lo, hi};
  if constexpr (DT == DT_F16) return __builtin_bit_cast(unsigned, __builtin_convertvector(x, f16x2));
  else return __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
}
template <int DT> __device__ __forceinline__ uint16_t to_out(float x) {
  if constexpr (DT == DT_F16) return __builtin_bit_cast(uint16_t, (_Float16)x);
  else return __builtin_bit_cast(uint16_t, (__bf16)x);
}

// One output element at byte offset `off` of C (fp32 results are stored as is).
template <int DT> __device__ __forceinline__ void store_out(float x, Rsrc rc, int off) {
  if constexpr (DT == DT_F32)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), rc, off, 0, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b16(to_out<DT>(x), rc, off, 0, 0);
}

// ---------------------------------------------------------------------------
// Tile order: logical tile ids are laid out so that the first
// floor(T/8)*8 ids dealt round-robin to the 8 XCDs land on one XCD in
// consecutive runs, then grouped by GROUP_M tile rows so neighbours share
// A rows and B columns in that XCD's L2.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void tile_coords(int t, const KArgs& p, int& tm, int& tn) {
  const int T = p.tiles_m * p.tiles_n;
  int logical = t;
  if (p.xcd_remap) {
    const int per = T >> 3;
    if (t < per * 8) logical = (t & 7) * per + (t >> 3);
  }
  const int gm = p.group_m;
  const int group_size = gm * p.tiles_n;
  const int group = logical / group_size;
  const int first_m = group * gm;
  const int rows_here = min(p.tiles_m - first_m, gm);
  const int in_group = logical - group * group_size;
  tm = first_m + in_group % rows_here;
  tn = in_group / rows_here;
}

// owner_of / locate (gdy_internal.h) with this workgroup's index.
__device__ __forceinline__ int owner_of(const KLaunch& L) { return owner_of(L, (int)blockIdx.x); }
__device__ __forceinline__ void locate(const KLaunch& L, int& gi, int& lwg, int& nwg) {
  locate(L, (int)blockIdx.x, gi, lwg, nwg);
}

// ---------------------------------------------------------------------------
// Element-wise add member (the non-GEMM that co-runs with GEMMs, Sec. 7.1):
// C = A + B over an M x N region of one type (bf16, fp16 or fp32), summed in
// fp32 and rounded once.  Its workgroup tile is kEwRows rows x 32 16-byte
// vectors whatever the block size, so an add has the same tile grid in its
// own kernel and inside a GEMM kernel's dispatch; a block of NT threads
// covers a tile in kEwRows * 32 / NT row passes and issues every load of the
// tile before the first sum.  Reads outside an operand's extent return 0
// through the buffer resource; stores are masked to the region.
// ---------------------------------------------------------------------------
constexpr int kEwRows = 32;
template <int DT> struct EwCols { static constexpr int v = 32 * 16 / ElemSize<DT>::v; };

template <int DT> __device__ __forceinline__ float ew_decode(unsigned bits);
template <> __device__ __forceinline__ float ew_decode<DT_BF16>(unsigned bits) {
  return __builtin_bit_cast(float, bits << 16);
}
template <> __device__ __forceinline__ float ew_decode<DT_F16>(unsigned bits) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}
template <> __device__ __forceinline__ float ew_decode<DT_F32>(unsigned bits) {
  return __builtin_bit_cast(float, bits);
}

// The thread's 16 bytes of one operand row: one vector load, or element by
// element where the base, pitch or item stride is not 16-byte aligned.
template <int ES>
__device__ __forceinline__ u32x4 ew_load(Rsrc r, int vec, int off) {
  if (vec) return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16 / ES; ++e) w[e * ES / 4] |= load_elem<ES>(r, off + e * ES) << ((e * ES * 8) & 31);
  return w;
}

template <int DT, int NT>
__device__ __forceinline__ void ew_add_tiles(const KArgs& p, int lwg, int nwg) {
  constexpr int ES = ElemSize<DT>::v;
  constexpr int VEC = 16 / ES;
  constexpr int RP = NT / 32;  // rows per pass
  constexpr int PASSES = kEwRows / RP;
  static_assert(PASSES >= 1 && kEwRows % RP == 0, "the block must tile the add's rows");
  Rsrc ra = make_rsrc(p.a, p.a_bytes);
  Rsrc rb = make_rsrc(p.b, p.b_bytes);
  Rsrc rc = make_rsrc(p.c, p.c_bytes);
  const int Mrows = (int)p.m, Ncols = (int)p.n;
  const int lda_b = (int)p.lda * ES, ldb_b = (int)p.ldb * ES, ldc_b = (int)p.ldc * ES;
  const int ntiles = p.tiles_m * p.tiles_n;
  const int total = ntiles * p.batch;
  const int r = threadIdx.x / 32, v = threadIdx.x % 32;
  for (int tb = lwg; tb < total; tb += nwg) {
    int t = tb;
    if (p.batch > 1) {
      const int item = tb / ntiles;
      t = tb - item * ntiles;
      ra = make_rsrc(p.a + item * p.stride_a, p.a_bytes);
      rb = make_rsrc(p.b + item * p.stride_b, p.b_bytes);
      rc = make_rsrc(p.c + item * p.stride_c, p.c_bytes);
    }
    const int row0 = (t / p.tiles_n) * kEwRows + r;
    const int col0 = (t % p.tiles_n) * EwCols<DT>::v + v * VEC;
    if (col0 >= Ncols) continue;
    u32x4 wa[PASSES], wb[PASSES];
#pragma unroll
    for (int s = 0; s < PASSES; ++s) {
      const int row = row0 + s * RP;
      if (row < Mrows) {
        wa[s] = ew_load<ES>(ra, p.a_vec, row * lda_b + col0 * ES);
        wb[s] = ew_load<ES>(rb, p.b_vec, row * ldb_b + col0 * ES);
      }
    }
    const bool whole = p.c_vec && col0 + VEC <= Ncols;  // two 8-byte stores
#pragma unroll
    for (int s = 0; s < PASSES; ++s) {
      const int row = row0 + s * RP;
      if (row >= Mrows) break;
      const int off = row * ldc_b + col0 * ES;
      u32x4 out = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const int sh = (e * ES * 8) & 31;
        const unsigned mask = ES == 4 ? 0xffffffffu : 0xffffu;
        const float x = ew_decode<DT>((wa[s][e * ES / 4] >> sh) & mask);
        const float y = ew_decode<DT>((wb[s][e * ES / 4] >> sh) & mask);
        if constexpr (DT == DT_F32) {
          out[e] = __builtin_bit_cast(unsigned, x + y);
        } else {
          out[e * ES / 4] |= (unsigned)to_out<DT>(x + y) << sh;
        }
      }
      if (whole) {
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{out[0], out[1]}, rc, off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{out[2], out[3]}, rc, off + 8, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          if (col0 + e >= Ncols) break;
          const int sh = (e * ES * 8) & 31;
          if constexpr (DT == DT_F32)
            __builtin_amdgcn_raw_buffer_store_b32(out[e], rc, off + e * ES, 0, 0);
          else
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(out[e * ES / 4] >> sh), rc, off + e * ES, 0, 0);
        }
      }
    }
  }
}

// An add member of any type run by a block of NT threads (a GEMM kernel's
// dispatch holds adds next to its GEMMs: KArgs::ew names their type).
template <int NT>
__device__ __forceinline__ void ew_member(const KArgs& p, int lwg, int nwg) {
  if (p.ew == DT_BF16) ew_add_tiles<DT_BF16, NT>(p, lwg, nwg);
  else if (p.ew == DT_F16) ew_add_tiles<DT_F16, NT>(p, lwg, nwg);
  else if (p.ew == DT_F32) ew_add_tiles<DT_F32, NT>(p, lwg, nwg);
}

// ---------------------------------------------------------------------------
// Split-K.  A GEMM with few tiles and a long K runs each tile as `split`
// work items over consecutive runs of `split_kt` K tiles, so more CUs stream
// its operands at once.  Each work item stores its unscaled fp32 partial
// into its run's row-major M x N plane of the workspace (plane (item *
// split + run), leading dimension N); a reduction kernel on the same stream
// then sums the planes in run order 0, 1, ..., scales, rounds and stores C.
// The kernel boundary orders the two: no atomics, no fences, no counters,
// and the sum does not depend on which run finished first.
// ---------------------------------------------------------------------------
// K range of split run s: the operand resources start at its first K tile
// and the GEMM's K shrinks to the run's length.
__device__ __forceinline__ int split_k0(const KArgs& p, int s, int bk) { return s * p.split_kt * bk; }

// The fp32 partial plane of run s of batch item `item`.
__device__ __forceinline__ float* split_plane(const KArgs& p, int item, int s) {
  return p.ws + ((size_t)item * p.split + s) * (size_t)p.m * (size_t)p.n;
}

// Reduction of the split planes of up to kMaxFused GEMMs (one launch per
// dispatch that split): 256 threads, 8 rows x 128 columns per tile, four
// consecutive columns per thread; C = round(scale * (P0 + P1 + ...)).
template <int OUT>
__global__ void __launch_bounds__(256) split_reduce(KLaunch L) {
  const int gi = owner_of(L);
  const KArgs& p = L.g[gi];
  const int wg0 = L.first[gi];
  const int nwg = L.first[gi + 1] - wg0;
  constexpr int OS = OUT == DT_F32 ? 4 : 2;
  const int M = (int)p.m, N = (int)p.n, S = p.split;
  const int tn = (N + 127) / 128, tm = (M + 7) / 8;
  const int ntiles = tm * tn, total = ntiles * p.batch;
  const int r = threadIdx.x / 32, v = threadIdx.x % 32;
  const int ldc_b = (int)p.ldc * OS;
  const size_t plane = (size_t)M * (size_t)N;
  for (int tb = (int)blockIdx.x - wg0; tb < total; tb += nwg) {
    const int item = tb / ntiles, t = tb - item * ntiles;
    const int row = (t / tn) * 8 + r, col0 = (t % tn) * 128 + v * 4;
    if (row >= M || col0 >= N) continue;
    const Rsrc rc = make_rsrc(p.c + item * p.stride_c, p.c_bytes);
    const float* P = p.ws + (size_t)item * S * plane + (size_t)row * N + col0;
    const int cols = min(4, N - col0);
    float acc[4];
    if (cols == 4 && (N & 3) == 0) {  // 16-byte aligned rows of the planes
      float4 x = *reinterpret_cast<const float4*>(P);
      acc[0] = x.x, acc[1] = x.y, acc[2] = x.z, acc[3] = x.w;
      for (int q = 1; q < S; ++q) {
        x = *reinterpret_cast<const float4*>(P + q * plane);
        acc[0] += x.x, acc[1] += x.y, acc[2] += x.z, acc[3] += x.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (e >= cols) break;
        acc[e] = P[e];
        for (int q = 1; q < S; ++q) acc[e] += P[q * plane + e];
      }
    }
    const int off = row * ldc_b + col0 * OS;
    bool stored = false;
    if constexpr (OUT != DT_F32) {  // four 16-bit outputs in one 8-byte store
      if (cols == 4 && p.c_vec) {
        u32x2 w;
        w[0] = to_out2<OUT>(acc[0] * p.scale, acc[1] * p.scale);
        w[1] = to_out2<OUT>(acc[2] * p.scale, acc[3] * p.scale);
        __builtin_amdgcn_raw_buffer_store_b64(w, rc, off, 0, 0);
        stored = true;
      }
    }
    if (!stored) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < cols) store_out<OUT>(acc[e] * p.scale, rc, off + e * OS);
    }
  }
}

}  // namespace gdy
