// lds_copy.h -- what the kernels that copy global memory straight into LDS
// share: counted waits, the copy itself, and the reads of MFMA operand
// fragments from K-contiguous and k-major tiles.
//
// LDS layouts (one K tile of an operand, 128 bytes of K):
//  * K-contiguous operand (A untransposed, B transposed): rows of 128 bytes of
//    K, no padding; the 16-byte chunk c of row r sits at position
//    c ^ ((r / 2) % 8), so the 16 rows of a fragment read hit 16 distinct bank
//    groups.
//  * k-major operand (B untransposed, A transposed): one row per k, chunks
//    swizzled by TileT::h, read with ds_read_b64_tr_b16 / ds_read_b64_tr_b8,
//    which transpose within each group of 16 lanes: with 16-bit data, output
//    lane i, element j comes from the address of lane i/4 + 4j, element i%4;
//    with 8-bit data, from lane i/8 + 2j, byte i%8.  Pointing lane L at row kb
//    + L/4 (kb + L/2) and columns 4*(L%4) (8*(L%2)) gives lane i consecutive k
//    of column i -- the MFMA operand layout.
// A copy writes 64 lanes x 16 bytes = 1 KiB of contiguous LDS per wave
// instruction; each lane picks the global chunk that belongs at its position.
#pragma once
#include "go_kernel.h"

namespace gdy {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;

// s_waitcnt with only the vector-memory counter constrained (gfx9 layout:
// vmcnt bits [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Buffer descriptor as four SGPRs (raw buffer, stride 0): the copies are
// issued from inline assembly so that the compiler neither tracks them nor
// adds its own waits (it would wait for every copy in flight before each
// barrier and LDS read, collapsing the ring to one stage).  Completion is
// tracked by hand with wait_vmcnt.
typedef int sdesc __attribute__((ext_vector_type(4)));

__device__ __forceinline__ sdesc make_sdesc(const void* base, int bytes) {
  const uint64_t a = (uint64_t)base;
  sdesc d;
  d[0] = (int)(uint32_t)a;
  d[1] = (int)((a >> 32) & 0xffffu);  // stride 0
  d[2] = bytes;
  d[3] = kRsrcWord3;
  return d;
}

constexpr int kOutOfRange = 0x7ffffff0;  // past any operand's extent: the copy writes zeros

// One 16-byte copy per lane: global byte `voffset` of `d` -> LDS address
// lds_addr + 16 * lane (lds_addr is wave-uniform).  The s_nop gives the wait
// states that the compiler does not insert in front of inline assembly: one
// after the write of M0 and, with SPILLS, five after a vector instruction that
// wrote a register of the descriptor.  Only kernels that keep scalars in lanes
// of vector registers (the build's resource report counts them as spilled
// SGPRs) have such writes; the five cost 2% of an 8192^3 GEMM.
template <bool SPILLS>
__device__ __forceinline__ void copy16_to_lds(sdesc d, const lds_u8* lds_base, int voffset) {
  const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds_base);
  if constexpr (SPILLS)
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "{m0}"(lds_addr), "v"(voffset), "s"(d)
                 : "memory");
  else
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "{m0}"(lds_addr), "v"(voffset), "s"(d)
                 : "memory");
}

// A workgroup-uniform value in scalar registers (nothing where the compiler
// knows; in the joint kernels, too large for it to follow the argument block's
// loads, it would keep the copies' descriptors in vector registers).
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x) {
  return (int64_t)(((uint64_t)(uint32_t)uniform((int)(x >> 32)) << 32) | (uint32_t)uniform((int)x));
}
template <class T> __device__ __forceinline__ T* uniform(T* p) { return (T*)uniform((int64_t)p); }
// The members of an argument block that the tile loops use, as scalars.
__device__ __forceinline__ KArgs uniform(const KArgs& q) {
  KArgs p = q;
  p.a = uniform(q.a), p.b = uniform(q.b), p.c = uniform(q.c);
  p.m = uniform((int)q.m), p.n = uniform((int)q.n), p.k = uniform((int)q.k);
  p.lda = uniform((int)q.lda), p.ldb = uniform((int)q.ldb), p.ldc = uniform((int)q.ldc);
  p.a_bytes = uniform(q.a_bytes), p.b_bytes = uniform(q.b_bytes), p.c_bytes = uniform(q.c_bytes);
  p.tiles_m = uniform(q.tiles_m), p.tiles_n = uniform(q.tiles_n), p.batch = uniform(q.batch);
  p.c_vec = uniform(q.c_vec), p.a_dma = uniform(q.a_dma), p.b_dma = uniform(q.b_dma);
  p.rows128 = uniform(q.rows128);
  p.split = uniform(q.split), p.split_kt = uniform(q.split_kt), p.ws = uniform(q.ws);
  p.stride_a = uniform(q.stride_a), p.stride_b = uniform(q.stride_b), p.stride_c = uniform(q.stride_c);
  return p;
}

// A member's arguments in its own kernel (as they are) and in a joint one.
template <bool JOINT> struct Args {
  const KArgs& v;
  __device__ __forceinline__ Args(const KArgs& a) : v(a) {}
};
template <> struct Args<true> {
  KArgs v;
  __device__ __forceinline__ Args(const KArgs& a) : v(uniform(a)) {}
};

// Workgroup barrier the compiler does not decorate with memory waits; the
// caller has already waited for its own copies.
__device__ __forceinline__ void barrier_nowait() { asm volatile("s_barrier" ::: "memory"); }

// ---- fragments of 16 x 16 MFMAs ---------------------------------------------
// Lane l covers row (column) l % 16 of the block and the K bytes
// [ks*4*FB + (l/16)*FB, +FB) of the tile.
template <int ES> struct FragT;  // fragment type by element size
template <> struct FragT<2> { typedef u32x4 T; static constexpr int FB = 16; };
template <> struct FragT<1> { typedef i32x8 T; static constexpr int FB = 32; };
// fp32: four K values of a 16 x 16 x 4 MFMA each; MFMA s of a K step takes the
// s-th value of every lane, K = 16*ks + 4*(l/16) + s for both operands.
template <> struct FragT<4> { typedef u32x4 T; static constexpr int FB = 16; };

__device__ __forceinline__ u32x4 lds_read16(const lds_u8* p) {
  return *(const __attribute__((address_space(3))) u32x4*)p;
}

// K-contiguous tile: per-lane offset at K step 0 (8-bit fragments are two
// chunks, e = 0 and 1); K step ks XORs 64*ks into it (8-bit tiles hold
// one step, the others two).
template <int ES> __device__ __forceinline__ int pk_lane(int lane, int e) {
  const int r = lane & 15, g = lane >> 4;
  const int c = ES == 1 ? 2 * g + e : g;
  return r * 128 + ((c ^ ((r >> 1) & 7)) << 4);
}
template <int ES>
__device__ __forceinline__ typename FragT<ES>::T pk_frag(const lds_u8* blk, int o0, int o1, int ks) {
  if constexpr (ES != 1) {
    return lds_read16(blk + (o0 ^ (64 * ks)));
  } else {
    const u32x4 lo = lds_read16(blk + o0), hi = lds_read16(blk + o1);
    i32x8 r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return r;
  }
}

// k-major tile of ROWS elements per k-row: 16-byte chunk c of row k at position
// c ^ h(k).  A transpose read takes, 32 lanes at a time, 16 columns of 4
// (16-bit: two chunks) or 8 (8-bit: one chunk) consecutive k-rows for two
// groups of lanes whose k differ by 8 (32).  Rows of 256 bytes and more all
// start on bank 0, shorter ones on the bank their k gives; h spreads those that
// share banks over different chunks (rows of 16 or 32 bytes, the transposed A
// of 16-row tiles, keep their order: two lanes to a bank).  fp32 needs no
// transpose: a read takes 16 columns of four k-rows 4 apart, one value a lane;
// their chunks go to different quarters of the banks.
template <int ES, int ROWS> struct TileT {
  static constexpr int RB = ROWS * ES;
  static constexpr int NCH = RB / 16;
  static constexpr int NHH = ES == 2 ? 2 : 4;  // reads of a fragment
  static_assert(RB >= 16 && RB <= 1024, "1 to 64 chunks per k-row");
  static __device__ __forceinline__ int h(int k) {
    if constexpr (ES == 4) {
      return (4 * ((k >> 2) & 3)) & (NCH - 1);
    } else if constexpr (RB < 64) {
      return 0;
    } else if constexpr (ES == 2) {
      if constexpr (RB >= 256) return (4 * (k & 3)) ^ (2 * ((k >> 3) & 1));
      else if constexpr (RB == 128) return (2 * ((k >> 1) & 1)) ^ (4 * ((k >> 3) & 1));
      else return 2 * ((k >> 3) & 1);
    } else {
      if constexpr (RB >= 256) return (2 * (k & 7)) ^ ((k >> 5) & 1);
      else if constexpr (RB == 128) return (2 * ((k >> 1) & 3)) ^ ((k >> 5) & 1);
      else return (2 * ((k >> 2) & 1)) ^ ((k >> 5) & 1);
    }
  }
  static __device__ __forceinline__ int addr(int k, int col) {
    const int byte = col * ES;
    return k * RB + (((byte >> 4) ^ h(k)) << 4) + (byte & 15);
  }
  // per-lane offset of sub-read hh of the 16-column fragment at col0, K step 0
  static __device__ __forceinline__ int lane_off(int lane, int col0, int hh) {
    const int L = lane & 15, kb = (lane >> 4) * (FragT<ES>::FB / ES);
    if constexpr (ES == 4) return addr(kb + hh, col0 + L);
    else if constexpr (ES == 2) return addr(kb + 4 * hh + (L >> 2), col0 + 4 * (L & 3));
    else return addr(kb + 8 * hh + (L >> 1), col0 + 8 * (L & 1));
  }
  // the fragment at K step ks (h does not change from one to the next)
  static __device__ __forceinline__ typename FragT<ES>::T frag(const lds_u8* tile, const int (&off)[NHH], int ks) {
    typename FragT<ES>::T r;
#pragma unroll
    for (int hh = 0; hh < NHH; ++hh) {
      if constexpr (ES == 4) {
        r[hh] = *(const __attribute__((address_space(3))) unsigned*)(tile + ks * 16 * RB + off[hh]);
        continue;
      }
      i32x2 w;
      if constexpr (ES == 2)
        w = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                          (__attribute__((address_space(3))) s16x4*)(tile + ks * 32 * RB + off[hh])));
      else
        w = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2*)(tile + off[hh]));
      r[2 * hh] = w[0];
      r[2 * hh + 1] = w[1];
    }
    return r;
  }
};

// The rounded BM x BN tile in LDS at `out` (rows of PITCH bytes) to C, all
// threads of the workgroup: 16 bytes a lane, or single elements where C's rows
// have no 8-byte alignment.  rows, cols: what of the tile lies inside C; off:
// its first byte.
template <int BN, int NT, int PITCH>
__device__ __forceinline__ void store_tile(const lds_u8* out, Rsrc rc, int off, int ldc_b, int rows, int cols,
                                           bool vec, int tid) {
  constexpr int LPR = BN / 8;  // lanes per row
  if (vec) {
    const int c8 = (tid % LPR) * 8;
    const int left = cols - c8;  // columns from this lane's first one
#pragma unroll 4
    for (int r = tid / LPR; r < rows; r += NT / LPR) {
      const u32x4 v = lds_read16(out + r * PITCH + c8 * 2);
      const int o = off + r * ldc_b + c8 * 2;
      if (left >= 8) {
        __builtin_amdgcn_raw_buffer_store_b128(v, rc, o, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e < left)
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(v[e / 2] >> (16 * (e & 1))), rc, o + 2 * e, 0, 0);
      }
    }
  } else {
    const int lane = tid & 63;
    for (int r = tid / 64; r < rows; r += NT / 64)
#pragma unroll
      for (int e = 0; e < BN / 64; ++e) {
        const int c = e * 64 + lane;
        if (c < cols)
          __builtin_amdgcn_raw_buffer_store_b16(
              *(const __attribute__((address_space(3))) uint16_t*)(out + r * PITCH + c * 2), rc,
              off + r * ldc_b + c * 2, 0, 0);
      }
  }
}

}  // namespace gdy
