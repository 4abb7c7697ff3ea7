// kernels_list.h -- the GO-Kernel catalogue: macro tiles x layouts for one
// input type.  Expanded once per type by the kernels_*.hip units, which
// define GDY_DT and GDY_DTNAME before including it.
//
// Tiles span the axes the tuner chooses from: large tiles (more LDS reuse,
// fewer workgroups) down to 16-row tiles for skinny GEMMs; 4 or 8 waves.
//
// Tiles above 128 x 128 (the host fills their kernels in: a null function):
// * 16- and 8-bit types, 256 x 256: GEMMs whose operands take copies run on the
//   alternating kernel (which only needs whole 16-byte chunks of K), others as
//   128 x 128 tiles of the joint kernel.  A 256 x 256 tile's accumulators leave
//   no registers for the unaligned way (it spilled 26 to 160; (1290, 3000, 1000)
//   bf16 34 us, on 128 x 128 tiles 20).
// * fp32: as 128 x 128 tiles.  Its MFMAs are 16 times slower than bf16 ones, so
//   LDS and L2 feed small tiles too, and those fill the chip better: the eight
//   GEMMs of a tensor-sliced layer took 4.87 ms on 256 x 256 and 3.87 on
//   256 x 128 tiles, 3.44 on 128 x 128; 4096^3 988, 1042 and 988 us.
#if GDY_DT32
#define GDY_KERNEL_LARGE(DT, DTNAME, TA, TB, LAYOUT, BM, BN, WM, WN)                      \
  {DTNAME "_" LAYOUT "_" #BM "x" #BN "_w" #WM "x" #WN "_m32", DT, TA, TB, BM, BN,          \
   ::gdy::UCfg<DT, 128, 128, 2, 2, 2>::BK, WM * WN, 16, 2 * (BM + BN) * 128, nullptr, 0, 0, \
   nullptr, 1, ::gdy::joint_code(TA, TB, BM, BN), 128, 128}
#define GDY_KERNEL_256(DT, DTNAME, TA, TB, LAYOUT) GDY_KERNEL_LARGE(DT, DTNAME, TA, TB, LAYOUT, 256, 256, 2, 4)
#else
#define GDY_KERNEL_LARGE(DT, DTNAME, TA, TB, LAYOUT, BM, BN, WM, WN)                      \
  GDY_KERNEL_U(DT, DTNAME, TA, TB, LAYOUT, BM, BN, WM, WN, 32)
#define GDY_KERNEL_256(DT, DTNAME, TA, TB, LAYOUT)                                       \
  {DTNAME "_" LAYOUT "_256x256_w2x4_m32", DT, TA, TB, 256, 256, ::gdy::PCfg<DT>::BK, 8,   \
   16, ::gdy::kPLds, nullptr, 0, 0, nullptr, 2, 2 * TA + TB, 256, 256}
#endif
#define GDY_TILES(L, TA, TB)                                   \
  GDY_KERNEL_256(GDY_DT, GDY_DTNAME, TA, TB, L),                 \
  GDY_KERNEL_LARGE(GDY_DT, GDY_DTNAME, TA, TB, L, 256, 128, 2, 2), \
  GDY_KERNEL_LARGE(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 256, 2, 2), \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 128, 2, 2, 32), \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 64, 256, 1, 4, 32),  \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 64, 128, 1, 4, 32),  \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 64, 64, 2, 2, 32),   \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 32, 256, 1, 4, 32),  \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 32, 128, 1, 4, 32),  \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 16, 256, 1, 4, 16),  \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 16, 128, 1, 4, 16),  \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 16, 64, 1, 4, 16)

// Transposed-A layouts carry a smaller set: weight gradients, which have them, are
// large in both dimensions and run on the 256 x 256 and 128 x 128 kernels.
#define GDY_TILES_SMALL(L, TA, TB)                             \
  GDY_KERNEL_256(GDY_DT, GDY_DTNAME, TA, TB, L),                 \
  GDY_KERNEL_LARGE(GDY_DT, GDY_DTNAME, TA, TB, L, 256, 128, 2, 2), \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 128, 2, 2, 32), \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 64, 64, 2, 2, 32),   \
  GDY_KERNEL_U(GDY_DT, GDY_DTNAME, TA, TB, L, 16, 64, 1, 4, 16)

static const ::gdy::KernelDesc kTable[] = {
    GDY_TILES("nn", 0, 0),
    GDY_TILES("nt", 0, 1),
    GDY_TILES_SMALL("tn", 1, 0),
    GDY_TILES_SMALL("tt", 1, 1),
};
