// go_kernel_u.h -- the GO-Kernels for tiles below 256 x 256, for operands of any
// size and alignment, and for fp32.
//
// Both operands lie in LDS in the layouts of lds_copy.h, and each gets there by
// one of two ways, chosen per GEMM:
//  * copies: base, pitch and item stride multiples of 16 bytes (and, for a
//    K-contiguous operand, K whole 16-byte chunks): direct global -> LDS
//    copies; chunks past K are sent out of range and read as zeros;
//  * registers: anything else.  A lane loads the five dwords around its 16
//    bytes (dword-aligned: what a buffer load needs), shifts them into place
//    with v_alignbit, zeroes what lies past K and writes the chunk to the same
//    place of the same layout.  K-major operands stay k-major: the transpose
//    is left to the LDS reads.
// The direct kernels (_dS) have the first way only, with a ring of S stages; the
// others (_m32, _m16), which the planner binds where K is no whole number of K
// tiles or an alignment is missing, have both and two stages.
//
// One barrier per K tile.  Direct: S - 1 tiles are in flight while one is
// computed.  Both ways: tile kt+1 goes to LDS while kt is computed, and in the
// register way tile kt+2 is being loaded, so a load has a whole tile's time to
// arrive.  Waves read a tile's fragments and issue its MFMAs; the other
// workgroup of the CU fills the gaps (tiles of up to 64 KiB of LDS).  Prefetching
// fragments across the barrier is slower, also where a workgroup has the CU to
// itself: the compiler moves them between the register files ((512, 6144, 12288)
// bf16 on 128 x 128, four stages, 122 us, 111 without; 4096^3, two stages, 152 and
// 140).  16 x 16 MFMAs (less energy a flop than 32 x 32); the rounded tile leaves
// through LDS as whole rows.
// Unaligned operands, on the kernels with element loads and register
// transposes before and on these: 2 x (509, 2047, 1021) fp16 on 64 x 64 tiles
// 55 and 19 us; K tails, 2 x (1000, 2000, 1000) bf16 on 128 x 128: 31 and 18 us.
#pragma once
#include "go_kernel_p.h"

namespace gdy {

// One operand of a tile: ROWS rows (or columns) x 128 bytes of K, KC:
// K-contiguous.  Lane `lane` of wave `wave` owns the chunks at LDS bytes
// (wave + NW*j)*1024 + lane*16 in both ways.
template <int ES, bool KC, int ROWS, int NW, bool SPILLS> struct Operand {
  static constexpr int BLOCKS = ROWS / 8;                   // 1 KiB copies of a K tile
  static constexpr int N = BLOCKS < NW ? 1 : BLOCKS / NW;   // chunks per lane
  static constexpr bool ALL = BLOCKS >= NW;                 // every wave takes part (16-row tiles: two do)
  static constexpr int BK = 128 / ES;
  static_assert(ROWS % 8 == 0 && (BLOCKS < NW || BLOCKS % NW == 0), "whole copies per wave");
  typedef TileT<ES, ROWS> T;
  const uint8_t* base;  // of the item and K run, down to a dword
  int bytes;            // from base to the end of the dword that holds the operand's last byte
  int step;             // bytes from one K tile to the next
  int jstep;            // bytes between this lane's chunks (K-contiguous)
  int off[KC ? 1 : N];  // byte offset of the lane's chunk(s) in K tile 0
  int kpos[KC ? 1 : N]; // K-contiguous: K byte of the chunk; k-major: its k
  u32x4 lo[N];
  unsigned hi[N];

  // extent: the operand's bytes from p on (items of a batch and K runs start at
  // any alignment, so the rounding up to whole dwords is this item's own)
  __device__ __forceinline__ void init(const uint8_t* p, int extent, int ld_b, int row0, int wave, int lane) {
    const int mis = (int)((uintptr_t)p & 3);
    base = p - mis;
    bytes = (extent + mis + 3) & ~3;
    step = KC ? 128 : BK * ld_b;
    jstep = 8 * NW * ld_b;
    if constexpr (KC) {
      const int r = wave * 8 + lane / 8;  // the swizzle of row r + 8*NW*j is that of row r (8*NW/2 = 0 mod 8)
      const int c = (lane & 7) ^ ((r >> 1) & 7);
      off[0] = (row0 + r) * ld_b + c * 16 + mis;
      kpos[0] = c * 16;
    } else {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int q = (wave + NW * j) * 64 + lane;
        const int k = q / T::NCH;
        off[j] = k * ld_b + row0 * ES + ((q % T::NCH) ^ T::h(k)) * 16 + mis;
        kpos[j] = k;
      }
    }
  }
  __device__ __forceinline__ int at(int j) const { return KC ? off[0] + j * jstep : off[KC ? 0 : j]; }

  __device__ __forceinline__ void copy(int kt, int kbytes, lds_u8* dst, int wave) const {
    if (!ALL && wave >= BLOCKS) return;
    const sdesc d = make_sdesc(base + (int64_t)kt * step, bytes - kt * step);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      int o = at(j);
      if constexpr (KC) o = kpos[0] < kbytes - kt * 128 ? o : kOutOfRange;
      copy16_to_lds<SPILLS>(d, dst + (wave + NW * j) * 1024, o);
    }
  }
  __device__ __forceinline__ void load(int kt, int wave) {
    if (!ALL && wave >= BLOCKS) return;
    const Rsrc r = make_rsrc(base + (int64_t)kt * step, bytes - kt * step);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int o = at(j) & ~3;
      lo[j] = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
      hi[j] = __builtin_amdgcn_raw_buffer_load_b32(r, o + 16, 0, 0);
    }
  }
  // K: elements of the run
  __device__ __forceinline__ void store(int kt, int K, lds_u8* dst, int wave, int lane) const {
    if (!ALL && wave >= BLOCKS) return;
    const int left = K - kt * BK;  // elements of K from this tile on
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const unsigned sh = (unsigned)(at(j) & 3) * 8;
      u32x4 v;
#pragma unroll
      for (int w = 0; w < 4; ++w) v[w] = __builtin_amdgcn_alignbit(w < 3 ? lo[j][w + 1] : hi[j], lo[j][w], sh);
      if (left < BK) {  // the last, partial tile
        if constexpr (KC) {
          const int nv = left * ES - kpos[0];  // bytes of this chunk below K
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int b = nv - 4 * w;
            v[w] &= b >= 4 ? 0xffffffffu : b <= 0 ? 0u : (1u << (8 * b)) - 1u;
          }
        } else if (kpos[KC ? 0 : j] >= left) {
          v = u32x4{0u, 0u, 0u, 0u};
        }
      }
      *(__attribute__((address_space(3))) u32x4*)(dst + (wave + NW * j) * 1024 + lane * 16) = v;
    }
  }
};

template <int DT, int BM, int BN, int WM, int WN, int STAGES> struct UCfg {
  static constexpr int ES = ElemSize<DT>::v;
  static constexpr int BK = 128 / ES;
  static constexpr int NW = WM * WN;
  static constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
  static constexpr int NKS = 128 / (4 * FragT<ES>::FB);  // MFMA K steps per tile
  static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int PITCH = BN * 2 + 16;  // of the rounded tile: a half wave's 16 rows on distinct banks
  static constexpr int OUT = ES == 4 ? 0 : BM * PITCH;  // fp32 results leave from the accumulators
  static constexpr int LDS = STAGES * STAGE > OUT ? STAGES * STAGE : OUT;
  static_assert(BM % (WM * 16) == 0 && BN % (WN * 16) == 0, "wave tile must hold whole 16 x 16 blocks");
  static_assert(LDS <= 160 * 1024, "LDS budget");
};

// The tiles of one member: work items lwg, lwg + nwg, ... of p, by the whole
// workgroup, in the LDS at smem (UCfg::LDS bytes).  ANY: both ways, else
// copies only.  SPLIT: members may be split along K.
template <int DT, int TA, int TB, int BM, int BN, int WM, int WN, int STAGES, bool ANY, bool SPLIT, bool JOINT>
__device__ __forceinline__ void u_tiles(const KArgs& args, int lwg, int nwg, lds_u8* smem) {
  const Args<JOINT> own(args);
  const KArgs& p = own.v;
  if constexpr (JOINT) lwg = uniform(lwg), nwg = uniform(nwg);
  typedef UCfg<DT, BM, BN, WM, WN, STAGES> C;
  typedef Mma<DT, 16> M;
  typedef typename FragT<C::ES>::T Frag;
  typedef f32x4 Acc;
  typedef Operand<C::ES, TA == 0, BM, C::NW, ANY || JOINT> OpA;
  typedef Operand<C::ES, TB == 1, BN, C::NW, ANY || JOINT> OpB;
  constexpr int NHH = OpA::T::NHH;
  constexpr int WTM = BM / WM, WTN = BN / WN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int ntiles = p.tiles_m * p.tiles_n;
  const int lda_b = (int)p.lda * C::ES, ldb_b = (int)p.ldb * C::ES, ldc_b = (int)p.ldc * OutSize<DT>::v;
  const int Mrows = (int)p.m, Ncols = (int)p.n;
  const bool acopy = !ANY || p.a_dma, bcopy = !ANY || p.b_dma;
  const int a_extent = TA == 0 ? (Mrows - 1) * lda_b + (int)p.k * C::ES : ((int)p.k - 1) * lda_b + Mrows * C::ES;
  const int b_extent = TB == 1 ? (Ncols - 1) * ldb_b + (int)p.k * C::ES : ((int)p.k - 1) * ldb_b + Ncols * C::ES;

  const int kc0 = pk_lane<C::ES>(lane, 0), kc1 = pk_lane<C::ES>(lane, 1);
  int aoff[C::FM][NHH], boff[C::FN][NHH];
  if constexpr (TA == 1) {
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int hh = 0; hh < NHH; ++hh) aoff[i][hh] = OpA::T::lane_off(lane, wm * WTM + i * 16, hh);
  }
  if constexpr (TB == 0) {
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int hh = 0; hh < NHH; ++hh) boff[j][hh] = OpB::T::lane_off(lane, wn * WTN + j * 16, hh);
  }

  // work items: every tile of every item of a strided batch; in the split
  // twin, each in `split` K runs (split innermost)
  const int nsplit = SPLIT ? p.split : 1;
  const int total = ntiles * p.batch * nsplit;
  for (int tb = lwg; tb < total; tb += nwg) {
    const int s_run = SPLIT ? tb % nsplit : 0;
    const int tile_all = SPLIT ? tb / nsplit : tb;
    const int item = tile_all / ntiles;
    const int t = tile_all - item * ntiles;
    int K = (int)p.k;
    int64_t a_shift = 0, b_shift = 0;
    if (SPLIT && nsplit > 1) {  // this run's K range: operands start at its first K tile
      const int k0 = split_k0(p, s_run, C::BK);
      K = min(K - k0, p.split_kt * C::BK);
      a_shift = TA == 0 ? (int64_t)k0 * C::ES : (int64_t)k0 * lda_b;
      b_shift = TB == 1 ? (int64_t)k0 * C::ES : (int64_t)k0 * ldb_b;
    }
    const Rsrc rc = make_rsrc(p.c + item * p.stride_c, p.c_bytes);
    const int nk = (K + C::BK - 1) / C::BK;
    int tm, tn;
    tile_coords(t, p, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    OpA oa;
    OpB ob;
    oa.init(p.a + item * p.stride_a + a_shift, a_extent - (int32_t)a_shift, lda_b, m0, wave, lane);
    ob.init(p.b + item * p.stride_b + b_shift, b_extent - (int32_t)b_shift, ldb_b, n0, wave, lane);

    Acc acc[C::FN][C::FM];  // C^T blocks: [n block][m block]
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int r = 0; r < M::NACC; ++r) acc[j][i][r] = 0.f;

    // The MFMAs of the K tile at As; `between` runs once the first fragments
    // have been read.  The direct kernels read the fragments of every K step
    // before the first MFMA (the fences keep the reads there): left to itself the
    // compiler moves a step's reads in front of its own MFMAs, where each waits for
    // LDS with nothing to do.  128 x 128, two stages, bf16 nt: 4096^3 135 -> 121 us,
    // (1000, 8192, 8192) 130 -> 117; nothing slower.  The others read a step at a
    // time: the second step's registers cost them a resident workgroup.
    constexpr bool AHEAD = !ANY;
    auto compute = [&](const lds_u8* As, auto between) {
      const lds_u8* Bs = As + C::A_BYTES;
      auto read = [&](int ks, Frag (&af)[C::FM], Frag (&bf)[C::FN]) {
#pragma unroll
        for (int j = 0; j < C::FN; ++j) {
          if constexpr (TB == 1) bf[j] = pk_frag<C::ES>(Bs + (wn * WTN + j * 16) * 128, kc0, kc1, ks);
          else bf[j] = OpB::T::frag(Bs, boff[j], ks);
        }
#pragma unroll
        for (int i = 0; i < C::FM; ++i) {
          if constexpr (TA == 0) af[i] = pk_frag<C::ES>(As + (wm * WTM + i * 16) * 128, kc0, kc1, ks);
          else af[i] = OpA::T::frag(As, aoff[i], ks);
        }
      };
      auto mma = [&](const Frag (&af)[C::FM], const Frag (&bf)[C::FN]) {
#pragma unroll
        for (int s = 0; s < (C::ES == 4 ? 4 : 1); ++s)  // fp32: the four MFMAs of a K step
#pragma unroll
          for (int j = 0; j < C::FN; ++j)
#pragma unroll
            for (int i = 0; i < C::FM; ++i) {
              if constexpr (C::ES == 4) {
                const unsigned b = bf[j][s], a = af[i][s];  // copies: a bit cast of a vector's element takes its first
                acc[j][i] = M::run(__builtin_bit_cast(float, b), __builtin_bit_cast(float, a), acc[j][i]);
              } else {
                acc[j][i] = M::run(bf[j], af[i], acc[j][i]);
              }
            }
      };
      if constexpr (AHEAD) {
        Frag af[C::NKS][C::FM], bf[C::NKS][C::FN];
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
          read(ks, af[ks], bf[ks]);
          __builtin_amdgcn_sched_barrier(0);
          if (ks == 0) between();
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) mma(af[ks], bf[ks]);
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
          Frag af[C::FM], bf[C::FN];
          read(ks, af, bf);
          if (ks == 0) between();
          mma(af, bf);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    // Past this barrier the tile whose copies the wave has waited for is in LDS
    // for every wave, and every wave's reads of the tile before are done.
    auto sync = [&]() {
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __builtin_amdgcn_sched_barrier(0);
      barrier_nowait();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto copy_tile = [&](int kt, int stage) {
      lds_u8* st = smem + stage * C::STAGE;
      oa.copy(kt, K * C::ES, st, wave);
      ob.copy(kt, K * C::ES, st + C::A_BYTES, wave);
    };

    if (nk > 0) {
      if (ANY && (STAGES == 2 || !acopy || !bcopy)) {
        // tile kt to its stage (register way: the values loaded before), and
        // the loads of the tile after it
        auto stage_in = [&](int kt) {
          lds_u8* st = smem + (kt & 1) * C::STAGE;
          if (acopy) {
            oa.copy(kt, K * C::ES, st, wave);
          } else {
            oa.store(kt, K, st, wave, lane);
            if (kt + 1 < nk) oa.load(kt + 1, wave);
          }
          if (bcopy) {
            ob.copy(kt, K * C::ES, st + C::A_BYTES, wave);
          } else {
            ob.store(kt, K, st + C::A_BYTES, wave, lane);
            if (kt + 1 < nk) ob.load(kt + 1, wave);
          }
        };
        if (!acopy) oa.load(0, wave);
        if (!bcopy) ob.load(0, wave);
        stage_in(0);
        for (int kt = 0; kt < nk; ++kt) {
          wait_vmcnt<0>();
          sync();
          compute(smem + (kt & 1) * C::STAGE, [&]() {
            if (kt + 1 < nk) stage_in(kt + 1);
          });
        }
      } else {
        // ring: STAGES - 1 tiles in flight while one is computed
        constexpr int PER = OpA::N + OpB::N;  // copies of a wave per tile
        static_assert((ANY && STAGES == 2) || (OpA::ALL && OpB::ALL && (STAGES - 2) * PER < 64), "counted copies");
        wait_vmcnt<0>();  // the previous tile's stores
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s)
          if (s < nk) copy_tile(s, s);
        int cur = 0, free = STAGES - 1;  // stages of tile kt and of tile kt + STAGES - 1
        for (int kt = 0; kt < nk; ++kt) {
          const int after = min(STAGES - 2, nk - 1 - kt);  // tiles issued after tile kt
          if (STAGES >= 4 && after >= 2) wait_vmcnt<(STAGES >= 4 ? 2 * PER : 0)>();
          else if (STAGES >= 3 && after >= 1) wait_vmcnt<(STAGES >= 3 ? PER : 0)>();
          else wait_vmcnt<0>();
          sync();
          compute(smem + cur * C::STAGE, [&]() {
            if (kt + STAGES - 1 < nk) copy_tile(kt + STAGES - 1, free);
          });
          cur = cur + 1 == STAGES ? 0 : cur + 1;
          free = free + 1 == STAGES ? 0 : free + 1;
        }
      }
    }

    if constexpr (SPLIT) {
      if (nsplit > 1) {  // the run's unscaled fp32 partial into its plane
        float* P = split_plane(p, item, s_run);
        // (direct kernels: the others would lose a resident workgroup to its registers)
        constexpr bool ROWS = BM >= 64 && !ANY;
        bool whole_rows = false;
        if constexpr (ROWS) whole_rows = (Ncols & 3) == 0;
        if (whole_rows) {
          if constexpr (ROWS) {
            // Through LDS, 64 rows at a time, so that lanes store whole rows (up to 1
            // KiB of consecutive bytes an instruction; 64 in the accumulators' own
            // order, which tiles of fewer rows keep: (512, 1024, 4096) bf16 on 16 x
            // 128 tiles 26.6 us, 29.2 this way).  (200, 1024, 8192) bf16 nt, eight runs
            // on 128 x 128 tiles, with its reduction: 22.4 -> 20.3 us.
            constexpr int PP = BN * 4 + 16;  // row pitch: a half wave's 16 rows on distinct banks
            constexpr int HR = 64, LPR = BN / 4, NT = C::NW * 64;
            static_assert(HR * PP <= C::LDS, "the rows fit in the ring");
#pragma unroll
            for (int h = 0; h < BM / HR; ++h) {
              if (m0 + h * HR >= Mrows) break;
              __syncthreads();  // every wave has read its last fragments, or the rows before
#pragma unroll
              for (int i = 0; i < C::FM; ++i) {
                const int r = wm * WTM + i * 16 - h * HR;
                if (r < 0 || r >= HR) continue;
#pragma unroll
                for (int j = 0; j < C::FN; ++j)
                  *(__attribute__((address_space(3))) f32x4*)(smem + (r + (lane & 15)) * PP +
                                                              (wn * WTN + j * 16 + 4 * (lane >> 4)) * 4) = acc[j][i];
              }
              __syncthreads();
              const int c = (tid % LPR) * 4, rows = min(HR, Mrows - m0 - h * HR);
              float* dst = P + (size_t)(m0 + h * HR) * Ncols + n0 + c;
              if (n0 + c < Ncols) {
#pragma unroll 4
                for (int r = tid / LPR; r < rows; r += NT / LPR)
                  *reinterpret_cast<f32x4*>(dst + (size_t)r * Ncols) =
                      *(const __attribute__((address_space(3))) f32x4*)(smem + r * PP + c * 4);
              }
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < C::FN; ++j)
#pragma unroll
            for (int i = 0; i < C::FM; ++i) {
              const int row = m0 + wm * WTM + i * 16 + (lane & 15);
              const int col = n0 + wn * WTN + j * 16 + 4 * (lane >> 4);
              if (row >= Mrows) continue;
              float* dst = P + (size_t)row * Ncols + col;
              if (!ROWS && col + 4 <= Ncols && (Ncols & 3) == 0) {
                *reinterpret_cast<float4*>(dst) = make_float4(acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3]);
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (col + e < Ncols) dst[e] = acc[j][i][e];
              }
            }
        }
        __syncthreads();  // every wave is done with the stages before the next item refills them
        continue;
      }
    }

    // accumulator r of lane l is n = 4*(l/16) + r, m = l%16 of its block
    __syncthreads();  // every wave has read its last fragments
    const float s = p.scale;
    if constexpr (C::ES == 4) {  // 16 bytes a lane, 64 consecutive ones of 16 rows an instruction
#pragma unroll
      for (int j = 0; j < C::FN; ++j)
#pragma unroll
        for (int i = 0; i < C::FM; ++i) {
          const int row = m0 + wm * WTM + i * 16 + (lane & 15), col = n0 + wn * WTN + j * 16 + 4 * (lane >> 4);
          if (row >= Mrows) continue;
          const f32x4 x = acc[j][i] * s;
          const int off = row * ldc_b + col * 4;
          if (col + 4 <= Ncols) {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rc, off, 0, 0);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (col + e < Ncols) store_out<DT>(x[e], rc, off + 4 * e);
          }
        }
    }
    if constexpr (C::ES != 4) {
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int i = 0; i < C::FM; ++i) {
        const Acc& x = acc[j][i];
        const u32x2 v = {to_out2<DT>(x[0] * s, x[1] * s), to_out2<DT>(x[2] * s, x[3] * s)};
        *(__attribute__((address_space(3))) u32x2*)(smem + (wm * WTM + i * 16 + (lane & 15)) * C::PITCH +
                                                    (wn * WTN + j * 16 + 4 * (lane >> 4)) * 2) = v;
      }
    __syncthreads();
    store_tile<BN, C::NW * 64, C::PITCH>(smem, rc, m0 * ldc_b + n0 * 2, ldc_b, min(BM, Mrows - m0),
                                         min(BN, Ncols - n0), p.c_vec != 0, tid);
    }
    if (tb + nwg < total) __syncthreads();  // the next tile's copies overwrite the output rows
  }
}

template <int DT, int TA, int TB, int BM, int BN, int WM, int WN, int STAGES, bool ANY, bool SPLIT>
__global__ void __launch_bounds__(WM * WN * 64)
go_gemm_u(KLaunch L) {
  static_assert(!ANY || STAGES == 2, "the register way is a tile ahead of two stages");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[UCfg<DT, BM, BN, WM, WN, STAGES>::LDS];
  int gi, lwg, nwg;
  locate(L, gi, lwg, nwg);
  if (gi < 0) return;  // an idle slot of a placed dispatch
  const KArgs& p = L.g[gi];
  if (p.ew) ew_member<WM * WN * 64>(p, lwg, nwg);  // an element-wise add fused into this dispatch
  else u_tiles<DT, TA, TB, BM, BN, WM, WN, STAGES, ANY, SPLIT, false>(p, lwg, nwg, (lds_u8*)smem);
}

// ---------------------------------------------------------------------------
// Joint launches.  A group whose GEMMs bind several kernels of one type (tiles,
// layouts, alignments) would take a dispatch each, and a fork and join of a
// pool stream per dispatch cost 20-25 us, more than a short group's GEMMs.
// This kernel runs them in one grid: each member names its tile and layout
// (KArgs::code), and runs the same loop as in its own kernel.  A tile size
// changes where an element is computed, never its sum (one MFMA shape, K
// ascending), so results are those of the members' own kernels bit for bit.
// Registers and LDS are those of the largest member: two workgroups a CU.
// ---------------------------------------------------------------------------
// Codes: layout (2*TA + TB) * 8 + tile.  Tiles above 128 x 128 run as 128 x 128,
// wide ones as the 128-column (64 for 16 rows) tile of their height.
constexpr int joint_tile(int bm, int bn) {
  return bm >= 128 ? 0 : bm == 64 ? (bn == 64 ? 2 : 1) : bm == 32 ? 3 : 4;
}
constexpr int kJointBm[5] = {128, 64, 64, 32, 16}, kJointBn[5] = {128, 128, 64, 128, 64};
constexpr int joint_code(int ta, int tb, int bm, int bn) { return (2 * ta + tb) * 8 + joint_tile(bm, bn); }
constexpr int kJointLds = 80 * 1024;

template <int DT, int TA, int TB>
__device__ __forceinline__ void joint_tiles(const KArgs& p, int lwg, int nwg, lds_u8* smem) {
  switch (p.code & 7) {
    case 0: u_tiles<DT, TA, TB, 128, 128, 2, 2, 2, true, true, true>(p, lwg, nwg, smem); break;
    case 2: u_tiles<DT, TA, TB, 64, 64, 2, 2, 4, true, true, true>(p, lwg, nwg, smem); break;
    case 4: u_tiles<DT, TA, TB, 16, 64, 1, 4, 2, true, true, true>(p, lwg, nwg, smem); break;
    default:  // the catalogue has these for an untransposed A only
      if constexpr (TA == 0) {
        if ((p.code & 7) == 1) u_tiles<DT, TA, TB, 64, 128, 2, 2, 3, true, true, true>(p, lwg, nwg, smem);
        else u_tiles<DT, TA, TB, 32, 128, 1, 4, 4, true, true, true>(p, lwg, nwg, smem);
      }
  }
}

template <int DT>
__global__ void __launch_bounds__(256)
go_gemm_joint(KLaunch L) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem_raw[kJointLds];
  lds_u8* smem = (lds_u8*)smem_raw;
  int gi, lwg, nwg;
  locate(L, gi, lwg, nwg);
  if (gi < 0) return;
  const KArgs& p = L.g[gi];
  if (p.ew) {
    ew_member<256>(p, lwg, nwg);
    return;
  }
  switch (p.code >> 3) {
    case 0: joint_tiles<DT, 0, 0>(p, lwg, nwg, smem); break;
    case 1: joint_tiles<DT, 0, 1>(p, lwg, nwg, smem); break;
    case 2: joint_tiles<DT, 1, 0>(p, lwg, nwg, smem); break;
    default: joint_tiles<DT, 1, 1>(p, lwg, nwg, smem);
  }
}

}  // namespace gdy

// Catalogue entries.  _m32 / _m16: any operands (the names are those of the
// register-staged family, whose MFMA block they gave); _dS: direct copies only,
// S stages.
#define GDY_KERNEL_UX(DT, TA, TB, BM, BN, WM, WN, ST, ANY, DIRECT, NAME)                              \
  {NAME, DT, TA, TB, BM, BN, ::gdy::UCfg<DT, BM, BN, WM, WN, ST>::BK, WM * WN, 16,                   \
   ::gdy::UCfg<DT, BM, BN, WM, WN, ST>::LDS,                                                          \
   reinterpret_cast<const void*>(&::gdy::go_gemm_u<DT, TA, TB, BM, BN, WM, WN, ST, ANY, false>), DIRECT, 0, \
   reinterpret_cast<const void*>(&::gdy::go_gemm_u<DT, TA, TB, BM, BN, WM, WN, ST, ANY, true>),       \
   WM * WN == 4 ? 1 : 0, ::gdy::joint_code(TA, TB, BM, BN),                                           \
   ::gdy::kJointBm[::gdy::joint_tile(BM, BN)], ::gdy::kJointBn[::gdy::joint_tile(BM, BN)]}
#define GDY_KERNEL_U(DT, DTNAME, TA, TB, LAYOUT, BM, BN, WM, WN, MM)                                  \
  GDY_KERNEL_UX(DT, TA, TB, BM, BN, WM, WN, 2, true, 0,                                               \
                DTNAME "_" LAYOUT "_" #BM "x" #BN "_w" #WM "x" #WN "_m" #MM)
#define GDY_KERNEL_D(DT, DTNAME, TA, TB, LAYOUT, BM, BN, WM, WN, ST)                                  \
  GDY_KERNEL_UX(DT, TA, TB, BM, BN, WM, WN, ST, false, 1,                                             \
                DTNAME "_" LAYOUT "_" #BM "x" #BN "_w" #WM "x" #WN "_d" #ST)
