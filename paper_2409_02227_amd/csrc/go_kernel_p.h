// go_kernel_p.h -- the 256 x 256 GO-Kernel on two alternating wave groups.
//
// Same GEMM and storage reading as go_kernel.h, operands and LDS layouts as in
// lds_copy.h: 16-byte aligned bases, pitches and item strides, and K whole
// 16-byte chunks where it is contiguous.  Eight waves
// compute a tile, two per SIMD, one of each group (waves 0-3 and 4-7).  While
// one group issues the MFMAs of a quarter of its K tile, the other reads the
// fragments of its next quarter from LDS and issues its copies; a barrier ends
// each interval and the groups swap.  So a SIMD's matrix core always has a
// wave whose operands are in registers, and LDS reads, copy issue and barrier
// arrival run beside MFMAs instead of between them.
//
// What bounds it: with all-zero operands an 8192^3 bf16 GEMM runs at 1890-1910
// TFLOP/s, with random ones the chip lowers its clock and it runs at 1445-1515
// (over chips, layouts and values; fp8 3580-3700 and 2840-2915), so energy per
// flop sets the rate of a large GEMM.  That decides the MFMA: 16 x 16 blocks move
// half the accumulator registers per flop of 32 x 32 ones (8192^3, bf16, B stored
// N x K, one chip: 1445 against 1345 TFLOP/s; the direct loop with one barrier
// per K tile that this one replaced: 1275; fp8, K x N: 2840, 2770 and 2458).
//
// A K tile holds 128 bytes of K per row, as half tiles of 16 KiB: the rows
// 0-127 and 128-255 of A (A0, A1) and the columns 0-127 and 128-255 of B (B0,
// B1).  Wave (wm, wn) owns rows wm*64 .. +64 of each half of A and columns
// wn*32 .. +32 of each half of B: quadrants of 64 x 32, one per phase, each
// phase being [reads, copies, vmcnt(8), barrier, MFMAs, barrier].
//
// 256-row tiles, two K tiles in LDS:
//   phase 0: reads A0(kt)              copies B1(kt+1)           MFMAs A0 x B0
//   phase 1: reads B1(kt)              copies A1(kt+1)           MFMAs A0 x B1
//   phase 2: reads A1(kt)              copies B0(kt+2)           MFMAs A1 x B0
//   phase 3: reads B0(kt+1)            copies A0(kt+2)           MFMAs A1 x B1
// 128-row tiles (no A1; a GEMM's last tile row when it holds at most 128
// rows), three K tiles in LDS:
//   phase 0: reads A0(kt)              copies B0(kt+2), A0(kt+2) MFMAs A0 x B0
//   phase 1: reads B1(kt), B0(kt+1)    copies B1(kt+2)           MFMAs A0 x B1
//
// Why vmcnt(8) is the wait of every phase: whatever a phase reads, this wave
// issued at most 8 copies after the copies of it by the time the phase before
// ends its reads (256 rows: four phases of 2 copies; 128 rows: B1(kt), B0(kt+1)
// and A0(kt+1) have 8 or more copies behind them in the order above).  Group 1
// runs one barrier behind group 0, so the waits of both groups in phase p come
// before the barrier that group 0 passes before it reads for phase p+1: every
// wave's copies are there.
// Why no copy overwrites a half tile that is still read: reads of phase p are
// in registers before the MFMAs that use them end, in phase p or (B0) p+1; for
// group 1 that is three (five) barriers after group 0 began phase p.  The copy
// into the same place comes at least two phases (four barriers), for B0 three
// (six), after that.
// Copies past the last K tile read nothing (out of range) and keep the count.
#pragma once
#include "lds_copy.h"

namespace gdy {

constexpr int kPHalf = 16 * 1024;          // bytes of a half tile
constexpr int kPLds = 9 * kPHalf;          // 2 x (A0 A1 B0 B1), or 3 x (A0 B0 B1)
constexpr int kPOutRow = 528;              // row pitch of the rounded tile in LDS
static_assert(256 * kPOutRow <= kPLds, "the rounded tile fits in the ring");

template <int DT> struct PCfg {
  static constexpr int ES = ElemSize<DT>::v;
  static constexpr int BK = 128 / ES;
  static constexpr int NKS = 128 / (4 * FragT<ES>::FB);  // MFMA K steps per tile
};

// One operand's copies into half tiles; KC: K-contiguous, else k-major.
template <int ES, bool KC, bool SPILLS> struct PhaseCopy {
  int off[2][2];  // per-lane byte offsets of the wave's two copies of each half
  int kbyte;      // KC: first K byte of this lane's chunk within the tile
  int step;       // bytes from one K tile to the next
  __device__ __forceinline__ void init(int ld_b, int row0, int wave, int lane) {
    step = KC ? 128 : (128 / ES) * ld_b;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int blk = wave + 8 * j;
        if constexpr (KC) {
          const int r = blk * 8 + lane / 8;
          const int c = (lane & 7) ^ ((r >> 1) & 7);  // r/2 mod 8 is the same for both copies
          kbyte = c * 16;
          off[hf][j] = (row0 + hf * 128 + r) * ld_b + c * 16;
        } else {
          const int q = blk * 64 + lane;
          const int k = q / TileT<ES, 128>::NCH;
          const int c = (q % TileT<ES, 128>::NCH) ^ TileT<ES, 128>::h(k);
          off[hf][j] = k * ld_b + (row0 + hf * 128) * ES + c * 16;
        }
      }
  }
  // Half `hf` of K tile kt into `dst`.  The resource starts at the K tile:
  // k-major rows past K then lie past its extent.  K-contiguous chunks past K
  // are sent out of range, as are tiles past the last one.
  __device__ __forceinline__ void issue(const uint8_t* base, int bytes, int kt, int kbytes, int nk, int hf,
                                        lds_u8* dst, int wave) const {
    const bool live = kt < nk;
    const int shift = live ? kt * step : 0;
    const sdesc d = make_sdesc(base + shift, live ? bytes - shift : 0);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int o = off[hf][j];
      if constexpr (KC) o = kbyte < kbytes - kt * 128 ? o : kOutOfRange;
      copy16_to_lds<SPILLS>(d, dst + (wave + 8 * j) * 1024, o);
    }
  }
};

// The tiles of one member (work items lwg, lwg + nwg, ... of p), in the kPLds
// bytes at smem.
template <int DT, int TA, int TB, bool JOINT>
__device__ __forceinline__ void p_tiles(const KArgs& args, int lwg, int nwg, lds_u8* smem) {
  const Args<JOINT> own(args);
  const KArgs& p = own.v;
  if constexpr (JOINT) lwg = uniform(lwg), nwg = uniform(nwg);
  typedef PCfg<DT> C;
  typedef Mma<DT, 16> M;
  typedef typename FragT<C::ES>::T Frag;
  typedef typename M::Acc Acc;
  typedef TileT<C::ES, 128> PT;  // a k-major half tile
  constexpr int NHH = PT::NHH;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave >> 2;  // also the wave's group
  const int wn = wave & 3;
  const int ntiles = p.tiles_m * p.tiles_n;
  const int lda_b = (int)p.lda * C::ES, ldb_b = (int)p.ldb * C::ES, ldc_b = (int)p.ldc * 2;
  const int Mrows = (int)p.m, Ncols = (int)p.n;
  const int kbytes = (int)p.k * C::ES;
  const int nk = (int)((p.k + C::BK - 1) / C::BK);

  // per-lane LDS offsets of the fragments within a half tile
  const int kc0 = pk_lane<C::ES>(lane, 0), kc1 = pk_lane<C::ES>(lane, 1);
  int aoff[4][NHH], boff[2][NHH];
  if constexpr (TA == 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hh = 0; hh < NHH; ++hh) aoff[i][hh] = PT::lane_off(lane, wm * 64 + i * 16, hh);
  }
  if constexpr (TB == 0) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int hh = 0; hh < NHH; ++hh) boff[j][hh] = PT::lane_off(lane, wn * 32 + j * 16, hh);
  }

  const int total = ntiles * p.batch;
  for (int tb = lwg; tb < total; tb += nwg) {
    const int item = tb / ntiles;
    const int t = tb - item * ntiles;
    const uint8_t* abase = p.a + item * p.stride_a;
    const uint8_t* bbase = p.b + item * p.stride_b;
    const Rsrc rc = make_rsrc(p.c + item * p.stride_c, p.c_bytes);
    int tm, tn;
    tile_coords(t, p, tm, tn);
    const int m0 = tm * (p.rows128 ? 128 : 256), n0 = tn * 256;
    const bool half = p.rows128 || Mrows - m0 <= 128;  // a 128-row tile

    PhaseCopy<C::ES, TA == 0, JOINT> ca;
    PhaseCopy<C::ES, TB == 1, JOINT> cb;
    ca.init(lda_b, m0, wave, lane);
    cb.init(ldb_b, n0, wave, lane);

    Acc acc[2][2][2][4];  // [half of A][half of B][16-column block][16-row block], C^T blocks
#pragma unroll
    for (int x = 0; x < 32; ++x)
#pragma unroll
      for (int r = 0; r < M::NACC; ++r) acc[x >> 4][(x >> 3) & 1][(x >> 2) & 1][x & 3][r] = 0.f;

    Frag af[C::NKS][4], bf[2][C::NKS][2];
    auto read_a = [&](const lds_u8* S) {
#pragma unroll
      for (int ks = 0; ks < C::NKS; ++ks)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (TA == 0) af[ks][i] = pk_frag<C::ES>(S + (wm * 64 + i * 16) * 128, kc0, kc1, ks);
          else af[ks][i] = PT::frag(S, aoff[i], ks);
        }
    };
    auto read_b = [&](const lds_u8* S, int hf) {
#pragma unroll
      for (int ks = 0; ks < C::NKS; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if constexpr (TB == 1) bf[hf][ks][j] = pk_frag<C::ES>(S + (wn * 32 + j * 16) * 128, kc0, kc1, ks);
          else bf[hf][ks][j] = PT::frag(S, boff[j], ks);
        }
    };
    // the second half of a phase: swap with the other group, MFMAs, swap back
    auto mma = [&](int ha, int hb) {
      wait_vmcnt<8>();
      __builtin_amdgcn_sched_barrier(0);
      barrier_nowait();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < C::NKS; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[ha][hb][j][i] = M::run(bf[hb][ks][j], af[ks][i], acc[ha][hb][j][i]);
      __builtin_amdgcn_sched_barrier(0);
      barrier_nowait();
      __builtin_amdgcn_sched_barrier(0);
    };

    if (nk > 0 && !half) {
      auto at = [&](int kt, int h) { return smem + (kt & 1) * (4 * kPHalf) + h * kPHalf; };  // h: A0 A1 B0 B1
      auto copy_a = [&](int kt, int hf) { ca.issue(abase, p.a_bytes, kt, kbytes, nk, hf, at(kt, hf), wave); };
      auto copy_b = [&](int kt, int hf) { cb.issue(bbase, p.b_bytes, kt, kbytes, nk, hf, at(kt, 2 + hf), wave); };
      wait_vmcnt<0>();  // the previous tile's stores
      copy_b(0, 0);
      copy_a(0, 0);
      copy_b(0, 1);
      copy_a(0, 1);
      copy_b(1, 0);
      copy_a(1, 0);
      wait_vmcnt<8>();
      barrier_nowait();
      read_b(at(0, 2), 0);
      if (wm) barrier_nowait();  // group 1 runs one barrier behind
      for (int kt = 0; kt < nk; ++kt) {
        read_a(at(kt, 0));
        copy_b(kt + 1, 1);
        mma(0, 0);
        read_b(at(kt, 3), 1);
        copy_a(kt + 1, 1);
        mma(0, 1);
        read_a(at(kt, 1));
        copy_b(kt + 2, 0);
        mma(1, 0);
        read_b(at(kt + 1, 2), 0);
        copy_a(kt + 2, 0);
        mma(1, 1);
      }
    } else if (nk > 0) {
      auto at = [&](int s, int h) { return smem + s * (3 * kPHalf) + h * kPHalf; };  // h: A0 B0 B1
      auto copy_a = [&](int kt, int s) { ca.issue(abase, p.a_bytes, kt, kbytes, nk, 0, at(s, 0), wave); };
      auto copy_b = [&](int kt, int s, int hf) {
        cb.issue(bbase, p.b_bytes, kt, kbytes, nk, hf, at(s, 1 + hf), wave);
      };
      wait_vmcnt<0>();
      copy_b(0, 0, 0);
      copy_a(0, 0);
      copy_b(0, 0, 1);
      copy_b(1, 1, 0);
      copy_a(1, 1);
      copy_b(1, 1, 1);
      wait_vmcnt<8>();
      barrier_nowait();
      read_b(at(0, 1), 0);
      if (wm) barrier_nowait();
      int s0 = 0, s1 = 1, s2 = 2;  // the LDS stages of K tiles kt, kt+1 and kt+2
      for (int kt = 0; kt < nk; ++kt) {
        read_a(at(s0, 0));
        copy_b(kt + 2, s2, 0);
        copy_a(kt + 2, s2);
        mma(0, 0);
        read_b(at(s0, 2), 1);
        read_b(at(s1, 1), 0);
        copy_b(kt + 2, s2, 1);
        mma(0, 1);
        const int s = s0;
        s0 = s1;
        s1 = s2;
        s2 = s;
      }
    }
    if (nk > 0) {
      if (!wm) barrier_nowait();
      wait_vmcnt<0>();  // no copy may land after the ring is reused or the workgroup has ended
      __syncthreads();
    }

    // Epilogue.  Blocks hold C^T: accumulator r of lane l is n = 4*(l/16) + r,
    // m = l%16.  The rounded tile goes through LDS (the ring is done with), so
    // that a wave stores whole rows: 16 bytes a lane, 512 consecutive bytes of
    // two rows an instruction, where the accumulators' own order gives 32.
    // The 528-byte row pitch keeps a half wave's 16 rows of 16 bytes on
    // distinct banks.
    const float s = p.scale;
#pragma unroll
    for (int ha = 0; ha < 2; ++ha) {
      if (ha && half) break;
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const Acc& x = acc[ha][hb][j][i];
            const int row = ha * 128 + wm * 64 + i * 16 + (lane & 15);
            const int col = hb * 128 + wn * 32 + j * 16 + 4 * (lane >> 4);
            const u32x2 v = {to_out2<DT>(x[0] * s, x[1] * s), to_out2<DT>(x[2] * s, x[3] * s)};
            *(__attribute__((address_space(3))) u32x2*)(smem + row * kPOutRow + col * 2) = v;
          }
    }
    __syncthreads();
    store_tile<256, 512, kPOutRow>(smem, rc, m0 * ldc_b + n0 * 2, ldc_b, min(half ? 128 : 256, Mrows - m0),
                                   min(256, Ncols - n0), p.c_vec != 0, (int)threadIdx.x);
    if (tb + nwg < total) __syncthreads();  // the next tile's copies overwrite the output rows
  }
}

template <int DT, int TA, int TB>
__global__ void __launch_bounds__(512)
go_gemm_p(KLaunch L) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kPLds];
  int gi, lwg, nwg;
  locate(L, gi, lwg, nwg);
  if (gi < 0) return;  // an idle slot of a placed dispatch
  const KArgs& p = L.g[gi];
  if (p.ew) ew_member<512>(p, lwg, nwg);  // an element-wise add fused into this dispatch
  else p_tiles<DT, TA, TB, false>(p, lwg, nwg, (lds_u8*)smem);
}

// Joint launch of 256 x 256 members of different layouts (KArgs::code =
// 2*TA + TB): one grid instead of a dispatch, fork and join per layout.
template <int DT>
__global__ void __launch_bounds__(512)
go_gemm_p_joint(KLaunch L) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem_raw[kPLds];
  lds_u8* smem = (lds_u8*)smem_raw;
  int gi, lwg, nwg;
  locate(L, gi, lwg, nwg);
  if (gi < 0) return;
  const KArgs& p = L.g[gi];
  if (p.ew) {
    ew_member<512>(p, lwg, nwg);
    return;
  }
  switch (p.code) {
    case 0: p_tiles<DT, 0, 0, true>(p, lwg, nwg, smem); break;
    case 1: p_tiles<DT, 0, 1, true>(p, lwg, nwg, smem); break;
    case 2: p_tiles<DT, 1, 0, true>(p, lwg, nwg, smem); break;
    default: p_tiles<DT, 1, 1, true>(p, lwg, nwg, smem);
  }
}

}  // namespace gdy

// Catalogue entries.  One kernel serves every 256 x 256 name of the direct
// catalogue (wave grid, stages: the loops it replaced; it was faster than each
// at every size tried, from (256, 4096, 1024) to 8192^3), so that GO tables
// that name them keep loading; KB is the name's K tile in bytes, which K must
// be a multiple of for the planner to bind it.  Its tiles exceed the split
// limit, so it has no split twin.
#define GDY_KERNEL_P(DT, DTNAME, TA, TB, LAYOUT, SUFFIX, KB)                                     \
  {DTNAME "_" LAYOUT "_256x256_" SUFFIX, DT, TA, TB, 256, 256, KB / ::gdy::ElemSize<DT>::v, 8, 16, \
   ::gdy::kPLds, reinterpret_cast<const void*>(&::gdy::go_gemm_p<DT, TA, TB>), 1, 0, nullptr,                     \
   2, 2 * TA + TB, 256, 256}
