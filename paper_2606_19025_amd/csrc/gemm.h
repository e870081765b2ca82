// Shared by the grouped-GEMM kernels (large bf16 tiles: gemm.hip, the others:
// gemm_tile.hip): the
// GEMM kinds, their arguments, the group table and the launch record.
#pragma once
#include <type_traits>

#include "common.h"

namespace moe {

// UP_FWD and DH_BWD are GU_FWD and DHH_BWD for the SiLU expert (one first
// projection W1 [H, d] instead of [Wg; Wu]).
enum GemmKind {
  GU_FWD = 0, DOWN_FWD = 1, DHH_BWD = 2, DX_BWD = 3, DWD = 4, DWGU = 5, UP_FWD = 6, DH_BWD = 7
};

template <int KIND>
struct Kind {
  static constexpr bool MRAG = KIND <= DX_BWD || KIND >= UP_FWD;  // ragged in M (else in K)
  static constexpr bool A_KC = MRAG;                                // A contiguous along k
  static constexpr bool B_KC = KIND <= DOWN_FWD || KIND == UP_FWD;  // B contiguous along k
};

struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  const void* aux;  // gu, read by the DHH_BWD epilogue
  void* out2;       // h, written by the GU_FWD epilogue
  const int32_t* offsets;
  long lda, ldb, ldc;
  long b_gs, c_gs;  // per-group strides (elements) of B and C
  long c_split;     // stride (elements) between the split-K partial outputs
  int n_groups, cap, M, N, K, H, accumulate;
  int ksplit;       // K-ragged kinds: each group's rows split in ksplit parts (0 = 1)
  // DOWN_FWD and DX_BWD (bf16): the kernel may cut K into up to ksplit_max
  // parts (its choice from the device-side group sizes); part p's fp32
  // partial goes to part + p c_split ([cap, N] each) and the choice to
  // *ksplit_used, for splitk_rows_reduce_kernel.  ksplit_max <= 1: no split.
  int ksplit_max;
  float* part;
  int* ksplit_used;
};

DEVI int clamp_row(int v, int cap) { return v < 0 ? 0 : (v > cap ? cap : v); }

// Group table of one set, staged in LDS once per block: the group offsets
// clamped to [0, cap] (c), their running maximum (b: group g of an M-ragged
// kind is rows [b[g], b[g+1])) and the number of m-tiles before group g (p).
constexpr int kMaxGroups = 256;
struct GroupTable {
  int c[kMaxGroups + 1], b[kMaxGroups + 1], p[kMaxGroups + 1];
  int uneven;  // (ragged in K) a group's tiles take over 1.25 times the average
};

DEVI int wave_incl_max(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v = max(v, u);
  }
  return v;
}
DEVI int wave_incl_sum(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  return v;
}

// Fill t from set a for m-tiles of BM rows (one wave; n_groups <= kMaxGroups).
// tile_rows: what a tile of a set ragged in K takes besides its group's rows (fill
// and epilogue, in rows).  (Found here, where the rows are at hand: a pass of
// its own over the table was slower.)
template <int BM>
DEVI void build_group_table(const GemmArgs& a, GroupTable& t, int tile_rows) {
  const int lane = threadIdx.x & 63;
  const int ng = a.n_groups;
  int run = 0;
  for (int g0 = 0; g0 <= ng; g0 += 64) {
    const int g = g0 + lane;
    const int c = g <= ng ? clamp_row(a.offsets[g], a.cap) : 0;
    int m = wave_incl_max(g <= ng ? c : 0);
    if (g0 > 0) m = max(m, run);
    if (g <= ng) {
      t.c[g] = c;
      t.b[g] = m;
    }
    run = __shfl(m, 63, 64);
  }
  WAIT_LGKMCNT(0);  // the wave's own table writes (lanes read their neighbours')
  int acc = 0;
  bool uneven = false;
  const float most = 1.25f * ((float)run + (float)tile_rows * (float)ng);
  for (int g0 = 0; g0 <= ng; g0 += 64) {
    const int g = g0 + lane;
    const int rows = g < ng ? t.b[g + 1] - t.b[g] : 0;
    const int tiles = (rows + BM - 1) / BM;
    uneven = uneven || __ballot((float)(rows + tile_rows) * (float)ng > most) != 0;
    const int inc = wave_incl_sum(tiles);
    if (g <= ng) t.p[g] = acc + inc - tiles;
    acc += __shfl(inc, 63, 64);
  }
  t.uneven = uneven;  // (the same from every lane)
  WAIT_LGKMCNT(0);
}

// Kernel argument of the GEMM kernels: up to kMaxSets sets of groups, each of
// GEMM kind KA or KB (kind_b[s] != 0), whose tiles share one
// launch - the routed and the merged shared experts of one kind, and in the
// backward two independent kinds (dHh with dW_d, dX with dW_gu), so that
// tiles of different lengths fill the CUs together, keep the CUs out of step
// (their epilogue stores do not all fall at once) and fill each other's last
// round.
constexpr int kMaxSets = 4;
struct GemmLaunch {
  GemmArgs s[kMaxSets];
  int kind_b[kMaxSets];
  int n_sets;
  int* counters;  // non-null: per-XCD tile counters (zero at launch) for dynamic dealing
};

// Timing names of the launches; the small tiles' end in _tile.
#define MOE_GEMM_NAMES(S)                                                                     \
  {"gemm_gu_fwd" S, "gemm_down_fwd" S, "gemm_dhh_bwd" S, "gemm_dx_bwd" S, "gemm_dwd" S,       \
   "gemm_dwgu" S, "gemm_up_fwd" S, "gemm_dh_bwd" S, "gemm_dhh_dwd" S, "gemm_dh_dwd" S,        \
   "gemm_dx_dwgu" S}
constexpr const char* kGemmNames[] = MOE_GEMM_NAMES("");
constexpr const char* kTileNames[] = MOE_GEMM_NAMES("_tile");
constexpr int gemm_name_index(int ka, int kb) {
  return ka == kb ? ka : ka == DHH_BWD ? 8 : ka == DH_BWD ? 9 : 10;
}

// Output tiles of the bf16 launches (fp32 ones choose by themselves).  TILE_32x64:
// launches of one kind only.
enum TileSize { TILE_256x256, TILE_64x128, TILE_64x64, TILE_32x64 };
// The small tiles (gemm_tile.hip): one launch over sets_a[0..na) of kind ka and
// sets_b[0..nb) of kind kb (kb == ka with nb = 0: one kind).
hipError_t run_gemm_tile(int bf16, int ka, int kb, const GemmArgs* sets_a, int na,
                         const GemmArgs* sets_b, int nb, TileSize size, hipStream_t s);

}  // namespace moe
