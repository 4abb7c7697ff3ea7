// kernels_d_list.h -- catalogue of direct (global->LDS copy) GO-Kernels for
// one input type; expanded by the kernels_d_*.hip units.  kernels_list.h holds
// the same tiles for the GEMMs the planner binds no direct kernel to (K not a
// multiple of the K tile, unaligned).
#define GDY_TILES_D(L, TA, TB)                                        \
  GDY_KERNEL_P(GDY_DT, GDY_DTNAME, TA, TB, L, "w2x4_d2", 128),        \
  GDY_KERNEL_P(GDY_DT, GDY_DTNAME, TA, TB, L, "w2x2_d2", 128),        \
  GDY_KERNEL_P(GDY_DT, GDY_DTNAME, TA, TB, L, "w2x4_d4h", 64),        \
  GDY_KERNEL_P(GDY_DT, GDY_DTNAME, TA, TB, L, "w2x2_d4h", 64),        \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 256, 128, 2, 2, 3),     \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 256, 2, 2, 3),     \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 128, 2, 2, 2),     \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 128, 2, 2, 4)

#define GDY_TILES_D_SMALL(L, TA, TB)                                  \
  GDY_KERNEL_P(GDY_DT, GDY_DTNAME, TA, TB, L, "w2x4_d2", 128),        \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 256, 128, 2, 2, 3),     \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 128, 128, 2, 2, 2)

// Small tiles with deep rings, for GEMMs whose few workgroups each walk a
// long K: there the time per K tile is the memory latency, and the ring keeps
// up to three tiles in flight where the two-stage kernel of the same tile keeps
// one.  64 x 128 has three stages under its four-stage name: two workgroups
// then share a CU ((512, 6144, 12288) bf16 161 -> 109 us, (64, 8192, 8192) 29.2
// and 30.5).  32-row tiles for 16-bit types only.
#if GDY_DT16
#define GDY_TILES_D_LAT32(L, TA, TB)                                  \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 32, 256, 1, 4, 3),      \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 32, 128, 1, 4, 4),
#else
#define GDY_TILES_D_LAT32(L, TA, TB)
#endif
#define GDY_TILES_D_LAT(L, TA, TB)                                    \
  GDY_TILES_D_LAT32(L, TA, TB)                                        \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 64, 256, 1, 4, 3),      \
  GDY_KERNEL_UX(GDY_DT, TA, TB, 64, 128, 2, 2, 3, false, 1,           \
                GDY_DTNAME "_" L "_64x128_w2x2_d4"),                  \
  GDY_KERNEL_D(GDY_DT, GDY_DTNAME, TA, TB, L, 64, 64, 2, 2, 4)

// A further 256 x 256 name of the 16-bit types.
#if GDY_DT16
#define GDY_TILES_D_WIDE(L, TA, TB) GDY_KERNEL_P(GDY_DT, GDY_DTNAME, TA, TB, L, "w4x4_d2", 128),
#else
#define GDY_TILES_D_WIDE(L, TA, TB)
#endif

static const ::gdy::KernelDesc kTableD[] = {
    GDY_TILES_D("nn", 0, 0),
    GDY_TILES_D("nt", 0, 1),
    GDY_TILES_D_WIDE("nn", 0, 0)
    GDY_TILES_D_WIDE("nt", 0, 1)
    GDY_TILES_D_SMALL("tn", 1, 0),
    GDY_TILES_D_SMALL("tt", 1, 1),
    GDY_TILES_D_LAT("nn", 0, 0),
    GDY_TILES_D_LAT("nt", 0, 1),
    GDY_KERNEL_D(GDY_DT, GDY_DTNAME, 1, 0, "tn", 64, 64, 2, 2, 4),
    GDY_KERNEL_D(GDY_DT, GDY_DTNAME, 1, 1, "tt", 64, 64, 2, 2, 4),
};
