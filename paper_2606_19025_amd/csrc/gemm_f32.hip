// Grouped GEMMs of fp32 layers on v_mfma_f32_16x16x4_f32 (fp32 products, fp32
// accumulation); the GEMM kinds and their operands are listed in gemm.hip.
//
// One block of 4 waves (2 x 2) per output tile of 32 MI x 32 NJ; a wave owns
// MI x NJ MFMA tiles of 16 x 16.  Operands pass through a ring of NS LDS
// stages of 32 k, filled by 16-byte global -> LDS DMA NS - 1 k-steps ahead:
// with registers between global memory and LDS, a k-step of a small GEMM (a
// few tiles, nothing else on the CU) waited out a whole memory latency.
// fp32 MFMA runs at 256 flop per clock and CU, so the LDS reads (8 to 16 bytes
// per clock and wave) and the L2 traffic of 64 x 64 tiles are far below their
// limits; the tile size is chosen for the number of blocks alone (run_kinds).
//
// Out-of-range rows, columns and k are read from a block of zeros; addresses
// are 64-bit, so operands may have any size.
//
// LDS layouts (per operand and stage), and which index an MFMA lane holds:
//  k-contiguous: row r holds 32 k (128 bytes); its 16-byte chunk c sits at
//    position c ^ ((r >> 1) & 7), so the 16 lanes of one read (consecutive
//    rows, one chunk) hit distinct bank groups.  Lane l reads 4 k of row
//    l % 16 of a 16-row tile: k = 16 q + 4 (l / 16) + e feeds MFMA e.
//  m/n-contiguous: row k holds the tile's 32 MI (32 NJ) indices.  Lane l reads
//    the MI consecutive indices MI (l % 16) + i of row 16 q + 4 (l / 16) + e:
//    index i belongs to the wave's MFMA tile i.
// The MFMA takes B as its first operand: register t of tile (i, j) is output
// column 4 (l / 16) + t of tile j, so 4 consecutive columns of a row end up in
// one lane for either layout of B, and every global access is 16 bytes.
#include "gemm.h"
#include "kernels.h"
#include "timing.h"

namespace moe {
namespace {

__device__ __attribute__((aligned(16))) const float kZeros[4] = {0.f, 0.f, 0.f, 0.f};

// lane l's 16 bytes at p -> LDS at base + 16 l (base wave-uniform).  The asm
// sets m0 and leaves the one wait state that an LDS DMA needs after it.
DEVI void dma16(const float* p, char* base) {
  const unsigned m0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_t*)base);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(m0)
               : "m0", "memory");
}

DEVI float dsilu_f(float g) {
  const float s = sigmoid_f(g);
  return s * (1.0f + g * (1.0f - s));
}

DEVI f32x4_t* vec(void* base, size_t i) {
  return reinterpret_cast<f32x4_t*>(static_cast<float*>(base) + i);
}
DEVI const f32x4_t* vec(const void* base, size_t i) {
  return reinterpret_cast<const f32x4_t*>(static_cast<const float*>(base) + i);
}

struct TileF32 {
  int g, row0, rows, m0, tile_n;
};

// Four consecutive output columns n .. n + 3 of tile row i (both in range).
template <int KIND>
DEVI void store_cols(const GemmArgs& a, const TileF32& t, int i, int n, f32x4_t v) {
  if constexpr (Kind<KIND>::MRAG) {
    const size_t m = (size_t)(t.row0 + i);
    if constexpr (KIND == DHH_BWD) {
      // dG = dHh U silu'(G), dU = dHh silu(G)
      const f32x4_t G = *vec(a.aux, m * 2 * a.H + n), U = *vec(a.aux, m * 2 * a.H + a.H + n);
      f32x4_t dG, dU;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dG[e] = v[e] * U[e] * dsilu_f(G[e]);
        dU[e] = v[e] * silu_f(G[e]);
      }
      *vec(a.C, m * 2 * a.H + n) = dG;
      *vec(a.C, m * 2 * a.H + a.H + n) = dU;
    } else if constexpr (KIND == DH_BWD) {
      const f32x4_t A = *vec(a.aux, m * a.H + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= dsilu_f(A[e]);
      *vec(a.C, m * a.ldc + n) = v;
    } else {
      *vec(a.C, m * a.ldc + n) = v;
      if constexpr (KIND == UP_FWD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = silu_f(v[e]);
        *vec(a.out2, m * a.H + n) = v;
      }
    }
  } else {
    f32x4_t* c = vec(a.C, (size_t)t.g * a.c_gs + (size_t)(t.m0 + i) * a.ldc + n);
    *c = a.accumulate ? *c + v : v;
  }
}

// Per-lane source of one 16-byte DMA piece: its address at k-step 0, its first
// k there and the k extent (0 for a row or column past the tile's).
struct Piece {
  const float* p;
  int k, k_end;
};

template <int KIND, int MI, int NJ, int NS>
DEVI void gemm_f32_tile(const GemmArgs& a, const TileF32& tl, char* lds) {
  using K_ = Kind<KIND>;
  constexpr int BM = 32 * MI, BN = 32 * NJ, BK = 32;
  constexpr int A_BYTES = BM * BK * 4, STAGE = (BM + BN) * BK * 4;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, g4 = lane >> 4;
  const float* A = static_cast<const float*>(a.A) + (size_t)tl.row0 * a.lda;
  const float* B = static_cast<const float*>(a.B) +
                   (K_::MRAG ? (size_t)tl.g * a.b_gs : (size_t)tl.row0 * a.ldb);
  const int Kd = K_::MRAG ? a.K : tl.rows;
  const int nk = (Kd + BK - 1) / BK;
  const int n0 = tl.tile_n * BN;

  // row of w_gate_up[g] (or of the second operand) behind tile column c; the
  // gate and up units of GU_FWD alternate in blocks of 8 NJ columns, half of a
  // wave's, so that a lane holds G and U of the same unit
  auto b_row = [&](int c, bool& ok) -> size_t {
    if constexpr (KIND == GU_FWD) {
      constexpr int HW = 8 * NJ;
      const int h = (n0 >> 1) + (c / (2 * HW)) * HW + c % HW;
      ok = h < a.H;
      return (size_t)((c / HW) & 1) * a.H + h;
    } else {
      ok = n0 + c < a.N;
      return (size_t)(n0 + c);
    }
  };
  // piece q of a k-contiguous operand: rows 8 q .. 8 q + 7
  auto piece_kc = [&](int q, const float* base, long ld, auto&& row_of) {
    const int r = q * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    bool ok;
    const size_t row = row_of(r, ok);
    return Piece{base + (ok ? row * ld : 0) + c * 4, c * 4, ok ? Kd : 0};
  };
  // piece q of an m/n-contiguous operand of R indices per row: 256 / R rows
  auto piece_mn = [&](int q, const float* base, long ld, int R, int i0, int end) {
    const int k = q * (256 / R) + lane / (R / 4);
    const int i = i0 + lane % (R / 4) * 4;
    return Piece{base + (size_t)k * ld + (i < end ? i : 0), k, i < end ? Kd : 0};
  };
  Piece pa[MI], pb[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int q = i * 4 + wave;
    if constexpr (K_::A_KC)
      pa[i] = piece_kc(q, A, a.lda, [&](int r, bool& ok) -> size_t { ok = r < tl.rows; return r; });
    else
      pa[i] = piece_mn(q, A, a.lda, BM, tl.m0, a.M);
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int q = j * 4 + wave;
    if constexpr (K_::B_KC) pb[j] = piece_kc(q, B, a.ldb, b_row);
    else pb[j] = piece_mn(q, B, a.ldb, BN, n0, a.N);
  }
  const long a_step = K_::A_KC ? BK : BK * a.lda, b_step = K_::B_KC ? BK : BK * a.ldb;
  // the next k-step's pieces into stage st (called once per k-step, in order)
  auto load = [&](int st) {
    char* la = lds + st * STAGE;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      dma16(pa[i].k < pa[i].k_end ? pa[i].p : kZeros, la + (i * 4 + wave) * 1024);
      pa[i].p += a_step;
      pa[i].k += BK;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      dma16(pb[j].k < pb[j].k_end ? pb[j].p : kZeros, la + A_BYTES + (j * 4 + wave) * 1024);
      pb[j].p += b_step;
      pb[j].k += BK;
    }
  };

  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // f[i][e]: fragment of MFMA tile i for the e-th MFMA of k-block q
  auto frags = [&](auto kc, auto ntag, const char* op, int w, int q, float (*f)[4]) {
    constexpr int N = decltype(ntag)::value;
    if constexpr (decltype(kc)::value) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int r = (w * N + i) * 16 + l16;
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(
            op + r * (BK * 4) + (((4 * q + g4) ^ ((r >> 1) & 7)) << 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) f[i][e] = v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        typedef __attribute__((__vector_size__(N * 4))) float vN;
        const vN v = *reinterpret_cast<const vN*>(
            op + ((16 * q + 4 * g4 + e) * 32 * N + (w * 16 + l16) * N) * 4);
#pragma unroll
        for (int i = 0; i < N; ++i) f[i][e] = v[i];
      }
    }
  };

#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < nk) load(p);
  for (int kt = 0; kt < nk; ++kt) {
    // this wave's pieces of k-step kt have landed (later ones may be in
    // flight); after the barrier everyone's have, and every wave is done with
    // the stage of k-step kt - 1, which k-step kt + NS - 1 takes
    wait_vm_groups<MI + NJ, NS - 2>(nk - 1 - kt);
    __syncthreads();
    if (kt + NS - 1 < nk) load((kt + NS - 1) % NS);
    const char* st = lds + (kt % NS) * STAGE;
#pragma unroll
    for (int q = 0; q < BK / 16; ++q) {
      float fa[MI][4], fb[NJ][4];
      frags(std::bool_constant<K_::A_KC>{}, std::integral_constant<int, MI>{}, st, wm, q, fa);
      frags(std::bool_constant<K_::B_KC>{}, std::integral_constant<int, NJ>{}, st + A_BYTES, wn, q, fb);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
    }
  }

  // epilogue, straight from the accumulators
  const int m_end = K_::MRAG ? tl.rows : a.M - tl.m0;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int r = K_::A_KC ? (wm * MI + i) * 16 + l16 : (wm * 16 + l16) * MI + i;
    if (r >= m_end) continue;
    if constexpr (KIND == GU_FWD) {
#pragma unroll
      for (int j = 0; j < NJ / 2; ++j) {
        const int h = (n0 >> 1) + wn * 8 * NJ + 16 * j + 4 * g4;
        if (h >= a.H) continue;
        const size_t m = (size_t)(tl.row0 + r);
        const f32x4_t G = acc[i][j], U = acc[i][j + NJ / 2];
        f32x4_t Hv;
#pragma unroll
        for (int e = 0; e < 4; ++e) Hv[e] = silu_f(G[e]) * U[e];
        *vec(a.C, m * 2 * a.H + h) = G;
        *vec(a.C, m * 2 * a.H + a.H + h) = U;
        *vec(a.out2, m * a.H + h) = Hv;
      }
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        int n;
        f32x4_t v;
        if constexpr (K_::B_KC) {
          n = n0 + (wn * NJ + j) * 16 + 4 * g4;
          v = acc[i][j];
        } else {  // the j-th group of four of the lane's 4 NJ consecutive columns
          n = n0 + (wn * 16 + 4 * g4) * NJ + 4 * j;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[i][(4 * j + e) % NJ][(4 * j + e) / NJ];
        }
        if (n < a.N) store_cols<KIND>(a, tl, r, n, v);
      }
    }
  }
}

constexpr int kXcds = 8;
constexpr int kBand = 8;  // m-tiles per band of the tile order

template <int KIND>
DEVI constexpr int cols_of(const GemmArgs& a) { return KIND == GU_FWD ? 2 * a.H : a.N; }

// Tile order as in the bf16 kernel: XCD x takes the x-th eighth of every set's
// tiles (blocks go to the XCDs round-robin by id), in bands of kBand m-tiles.
// The grid covers the largest number of tiles that the group sizes can give;
// blocks past the last tile end at once.
template <int KA, int KB, int MI, int NJ, int NS>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(GemmLaunch L) {
  constexpr int BM = 32 * MI, BN = 32 * NJ;
  constexpr int RING = NS * (BM + BN) * 128;
  static_assert(RING >= (int)sizeof(GroupTable) * kMaxSets, "the group tables share the ring");
  __shared__ __attribute__((aligned(1024))) char lds[RING];
  GroupTable* gtab = reinterpret_cast<GroupTable*>(lds);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wave < L.n_sets) build_group_table<BM>(L.s[wave], gtab[wave]);
  __syncthreads();
  const int xcd = blockIdx.x % kXcds;
  int i = blockIdx.x / kXcds;  // this block's tile among the XCD's
  int set = -1;
  TileF32 tl{};
  for (int q = 0; q < L.n_sets; ++q) {
    const GemmArgs& a = L.s[q];
    const bool kb = KA != KB && L.kind_b[q] != 0;
    const bool mrag = kb ? Kind<KB>::MRAG : Kind<KA>::MRAG;
    const int cols = kb ? cols_of<KB>(a) : cols_of<KA>(a);
    const int mt_g = mrag ? 0 : (a.M + BM - 1) / BM;
    const int m_tiles = __builtin_amdgcn_readfirstlane(mrag ? gtab[q].p[a.n_groups] : a.n_groups * mt_g);
    const int n_tiles = (cols + BN - 1) / BN;
    const long tot = (long)m_tiles * n_tiles;
    const long lo = tot * xcd / kXcds;
    const int cnt = (int)(tot * (xcd + 1) / kXcds - lo);
    if (i >= cnt) {
      i -= cnt;
      continue;
    }
    set = q;
    const long t = lo + i;
    const long band = t / ((long)kBand * n_tiles);
    const int first_m = (int)(band * kBand);
    const int band_m = min(kBand, m_tiles - first_m);
    const int r = (int)(t - band * kBand * n_tiles);
    const int mt = first_m + r % band_m;
    tl.tile_n = r / band_m;
    if (mrag) {
      int g = 0;  // the groups whose m-tiles all lie before this one
      for (int g0 = 0; g0 < a.n_groups; g0 += 64) {
        const int gg = g0 + lane;
        g += __builtin_popcountll(__ballot(gg < a.n_groups && gtab[q].p[gg + 1] <= mt));
      }
      g = __builtin_amdgcn_readfirstlane(g);
      tl.g = g;
      tl.row0 = gtab[q].b[g] + (mt - gtab[q].p[g]) * BM;
      tl.rows = min(BM, gtab[q].b[g + 1] - tl.row0);
      tl.m0 = 0;
    } else {
      tl.g = mt / mt_g;
      tl.m0 = mt % mt_g * BM;
      tl.row0 = gtab[q].c[tl.g];
      tl.rows = max(0, gtab[q].c[tl.g + 1] - tl.row0);
    }
    break;
  }
  tl.row0 = __builtin_amdgcn_readfirstlane(tl.row0);
  tl.rows = __builtin_amdgcn_readfirstlane(tl.rows);
  __syncthreads();  // the tables have been read: the ring takes their place
  if (set < 0) return;
  if constexpr (KA != KB) {
    if (L.kind_b[set]) {
      gemm_f32_tile<KB, MI, NJ, NS>(L.s[set], tl, lds);
      return;
    }
  }
  gemm_f32_tile<KA, MI, NJ, NS>(L.s[set], tl, lds);
}

template <int KIND, int MI, int NJ>
long max_tiles(const GemmArgs& a) {
  const long n = ceil_div(KIND == GU_FWD ? 2 * a.H : a.N, 32 * NJ);
  return n * (Kind<KIND>::MRAG ? (long)ceil_div(a.cap, 32 * MI) + std::min(a.n_groups, a.cap)
                               : (long)a.n_groups * ceil_div(a.M, 32 * MI));
}

template <int KA, int KB, int MI, int NJ>
long launch_tiles(const GemmArgs* sa, int na, const GemmArgs* sb, int nb) {
  long t = 0;
  for (int q = 0; q < na; ++q) t += max_tiles<KA, MI, NJ>(sa[q]);
  for (int q = 0; q < nb; ++q) t += max_tiles<KB, MI, NJ>(sb[q]);
  return t;
}

template <int KA, int KB, int MI, int NJ, int NS>
hipError_t launch(const GemmArgs* sa, int na, const GemmArgs* sb, int nb, hipStream_t s) {
  GemmLaunch L{};
  long blocks = 0;
  auto add = [&](const GemmArgs& a, int kb, long tiles) {
    L.s[L.n_sets] = a;
    L.kind_b[L.n_sets++] = kb;
    blocks += kXcds * ((tiles + kXcds - 1) / kXcds);
  };
  for (int q = 0; q < na; ++q) add(sa[q], 0, max_tiles<KA, MI, NJ>(sa[q]));
  for (int q = 0; q < nb; ++q) add(sb[q], 1, max_tiles<KB, MI, NJ>(sb[q]));
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffffL) return hipErrorInvalidConfiguration;
  MOE_TIMED((gemm_name<KA, KB>()), s,
            gemm_f32_kernel<KA, KB, MI, NJ, NS><<<(unsigned)blocks, 256, 0, s>>>(L));
  return hipGetLastError();
}

template <int KA, int KB>
hipError_t run_kinds(const GemmArgs* sa, int na, const GemmArgs* sb, int nb, hipStream_t s) {
  const long cus = num_cus();
  if (launch_tiles<KA, KB, 4, 4>(sa, na, sb, nb) >= 4 * cus)
    return launch<KA, KB, 4, 4, 2>(sa, na, sb, nb, s);
  if (launch_tiles<KA, KB, 2, 2>(sa, na, sb, nb) >= cus)
    return launch<KA, KB, 2, 2, 3>(sa, na, sb, nb, s);
  return launch<KA, KB, 1, 2, 4>(sa, na, sb, nb, s);
}

}  // namespace

hipError_t run_gemm_f32(int ka, int kb, const GemmArgs* sa, int na, const GemmArgs* sb, int nb,
                        hipStream_t s) {
#define MOE_KINDS(A, B) \
  if (ka == A && kb == B) return run_kinds<A, B>(sa, na, sb, nb, s)
  MOE_KINDS(GU_FWD, GU_FWD);
  MOE_KINDS(UP_FWD, UP_FWD);
  MOE_KINDS(DOWN_FWD, DOWN_FWD);
  MOE_KINDS(DHH_BWD, DWD);
  MOE_KINDS(DH_BWD, DWD);
  MOE_KINDS(DX_BWD, DWGU);
#undef MOE_KINDS
  return hipErrorInvalidValue;
}

}  // namespace moe
