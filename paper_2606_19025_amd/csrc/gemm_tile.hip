// Grouped GEMMs in small tiles: fp32 layers (v_mfma_f32_16x16x4_f32: fp32
// products, fp32 accumulation) and the bf16 launches that are too small for the
// 256 x 256 tiles (v_mfma_f32_16x16x32_bf16).  The GEMM kinds and their operands
// are listed in gemm.hip.
//
// One block of 4 waves (2 x 2) per output tile of 32 MI x 32 NJ; a wave owns
// MI x NJ MFMA tiles of 16 x 16.  Operands pass through a ring of NS LDS stages
// of 128 bytes of k (32 fp32, 64 bf16), filled by 16-byte global -> LDS DMA
// NS k-steps ahead: with registers between global memory and LDS, a k-step of a
// small GEMM (a few tiles, nothing else on the CU) waited out a whole memory
// latency.  Several blocks share a CU, so one's fill and epilogue pass under
// another's MFMAs.
// fp32 MFMA runs at 256 flop per clock and CU, so LDS reads and L2 traffic are
// far below their limits; what is left is the issue of the MFMAs: 70 % of their
// cycles are busy at 4096 rows, d = 1024, H = 1408 (forward and backward 0.98
// ms, 108 TFLOP/s; the 64 x 64 SIMT tiles before: about 14 TFLOP/s).
// bf16 is bound by LDS (a 64 x 128 tile reads and writes 1.5 to 2 times the
// bytes per flop of the large tiles' waves), so it loses at sizes that fill the
// CUs with large tiles, and wins below (choose_tiles in gemm.hip has the figures).
//
// k past the last are read from a block of zeros.  A piece's address is a 64-bit
// wave-uniform one plus a lane's 32-bit offset, or 64-bit per lane where that
// does not reach, so operands may have any size.
//
// LDS layouts (per operand and stage), and which index an MFMA lane holds:
//  k-contiguous: row r holds the stage's k (128 bytes); its 16-byte chunk c sits
//    at position c ^ ((r >> 1) & 7), so the 16 lanes of one read (consecutive
//    rows, one chunk) hit distinct bank groups.  Lane l reads 16 bytes of row
//    l % 16 of a 16-row tile: the 8 k of its bf16 MFMA, or (fp32) k = 16 q + 4
//    (l / 16) + e for MFMA e.
//  m/n-contiguous, bf16: row k holds the tile's 32 MI (or 32 NJ) indices in
//    32-byte chunks placed by mn_key; two transposing reads give a lane index l %
//    16 of a 16-index tile, 8 k.
//  m/n-contiguous, fp32: row k holds the tile's 32 MI (or 32 NJ) indices.  Lane l reads
//    the MI consecutive indices MI (l % 16) + i of row 16 q + 4 (l / 16) + e:
//    index i belongs to the wave's MFMA tile i.
// The MFMA takes B as its first operand: register t of tile (i, j) is output
// column 4 (l / 16) + t of tile j, so 4 consecutive columns of a row end up in
// one lane for either layout of B, and every fp32 access is 16 bytes.
#include "gemm.h"
#include "kernels.h"
#include "timing.h"

namespace moe {
namespace {

__device__ __attribute__((aligned(16))) const float kZeros[4] = {0.f, 0.f, 0.f, 0.f};

// A lane's 16 bytes -> LDS at base + 16 lane (base wave-uniform), from p, or from
// offset off (bytes) of a wave-uniform pointer.  The asm sets m0 and leaves the
// one wait state that an LDS DMA needs after it.
DEVI unsigned lds_offset(char* base) {
  return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_t*)base);
}
DEVI void dma16(const void* p, char* base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p),
               "s"(lds_offset(base))
               : "m0", "memory");
}
DEVI void dma16(const void* uniform, unsigned off, char* base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off),
               "s"(uniform), "s"(lds_offset(base))
               : "m0", "memory");
}

// Four consecutive fp32, eight bf16.
DEVI void put4(void* base, size_t i, f32x4_t v) {
  *reinterpret_cast<f32x4_t*>(static_cast<float*>(base) + i) = v;
}
DEVI f32x4_t get4(const void* base, size_t i) {
  return *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(base) + i);
}
DEVI void put8(void* base, size_t i, bf16x8_t v) {
  *reinterpret_cast<bf16x8_t*>(static_cast<bf16_t*>(base) + i) = v;
}
DEVI bf16x8_t get8(const void* base, size_t i) {
  return *reinterpret_cast<const bf16x8_t*>(static_cast<const bf16_t*>(base) + i);
}
// bf16: hardware exp2 and reciprocal (about 1 ulp of fp32), as in the large tiles
template <class T>
DEVI float sigmoid_t(float g) {
  if constexpr (sizeof(T) == 4) return sigmoid_f(g);
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * g));
}
template <class T>
DEVI float silu_t(float g) {
  if constexpr (sizeof(T) == 4) return silu_f(g);
  return g * sigmoid_t<T>(g);
}
template <class T>
DEVI float dsilu_t(float g) {
  const float s = sigmoid_t<T>(g);
  return s * (1.0f + g * (1.0f - s));
}

struct TileAt {
  int g, row0, rows, m0, tile_n;
};

// Four consecutive fp32 output columns n .. n + 3 of tile row i (both in range):
// rows of fp32 layers, weight gradients of either type.
template <int KIND>
DEVI void store_cols(const GemmArgs& a, const TileAt& t, int i, int n, f32x4_t v) {
  if constexpr (Kind<KIND>::MRAG) {
    const size_t m = (size_t)(t.row0 + i);
    if constexpr (KIND == DHH_BWD) {
      // dG = dHh U silu'(G), dU = dHh silu(G)
      const f32x4_t G = get4(a.aux, m * 2 * a.H + n), U = get4(a.aux, m * 2 * a.H + a.H + n);
      f32x4_t dG, dU;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dG[e] = v[e] * U[e] * dsilu_t<float>(G[e]);
        dU[e] = v[e] * silu_t<float>(G[e]);
      }
      put4(a.C, m * 2 * a.H + n, dG);
      put4(a.C, m * 2 * a.H + a.H + n, dU);
    } else if constexpr (KIND == DH_BWD) {
      const f32x4_t A = get4(a.aux, m * a.H + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= dsilu_t<float>(A[e]);
      put4(a.C, m * a.ldc + n, v);
    } else {
      put4(a.C, m * a.ldc + n, v);
      if constexpr (KIND == UP_FWD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = silu_t<float>(v[e]);
        put4(a.out2, m * a.H + n, v);
      }
    }
  } else {
    f32x4_t* c = reinterpret_cast<f32x4_t*>(static_cast<float*>(a.C) + (size_t)t.g * a.c_gs +
                                            (size_t)(t.m0 + i) * a.ldc + n);
    *c = a.accumulate ? *c + v : v;
  }
}

// bf16 m/n-contiguous rows of R indices: the 32-byte chunk c of row k sits at
// chunk c ^ mn_key<R>(k), so that the 8 rows (k0..k0+3 and k0+8..k0+11) a
// half-wave of transposing reads touches fall on distinct banks.
template <int R>
DEVI int mn_key(int k) {
  if constexpr (R >= 128) return (2 * (k & 3)) ^ ((k >> 3) & 1);
  if constexpr (R == 64) return (k & 2) ^ ((k >> 3) & 1);
  return (k >> 3) & 1;
}

// What a lane reads in one 16-byte DMA piece of a k-step: the elements at row r,
// column c of the operand's rows there; k is the (first) one's index along k.
struct Piece {
  int r, c, k;
};

template <class T, int KIND, int MI, int NJ, int NS>
DEVI void gemm_tile(const GemmArgs& a, const TileAt& tl, char* lds) {
  using K_ = Kind<KIND>;
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int V = 16 / sizeof(T);  // elements per 16 bytes
  constexpr int BM = 32 * MI, BN = 32 * NJ, BK = 8 * V;
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, g4 = lane >> 4;
  const T* A = static_cast<const T*>(a.A) + (size_t)tl.row0 * a.lda;
  const T* B = static_cast<const T*>(a.B) +
                   (K_::MRAG ? (size_t)tl.g * a.b_gs : (size_t)tl.row0 * a.ldb);
  const int Kd = K_::MRAG ? a.K : tl.rows;
  const int nk = (Kd + BK - 1) / BK;
  const int n0 = tl.tile_n * BN;

  // row of w_gate_up[g] (or of the second operand) behind tile column c; the
  // gate and up units of GU_FWD alternate in blocks of 8 NJ columns, half of a
  // wave's, so that a lane holds G and U of the same unit.  Columns past the
  // last (and rows past the group's, below) repeat a valid one: their outputs
  // are not stored.
  auto b_row = [&](int c) {
    if constexpr (KIND == GU_FWD) {
      constexpr int HW = 8 * NJ;
      const int h = (n0 >> 1) + (c / (2 * HW)) * HW + c % HW;
      return ((c / HW) & 1) * a.H + (h < a.H ? h : 0);
    } else {
      return min(n0 + c, a.N - 1);
    }
  };
  // piece q of a k-contiguous operand: rows 8 q .. 8 q + 7
  auto piece_kc = [&](int q, auto&& row_of) {
    const int r = q * 8 + (lane >> 3);
    const int c = ((lane & 7) ^ ((r >> 1) & 7)) * V;
    return Piece{row_of(r), c, c};
  };
  // piece q of an m/n-contiguous operand of R indices per row
  auto piece_mn = [&](auto r_tag, int q, int i0, int end) {
    constexpr int R = decltype(r_tag)::value, S = R / V;  // 16-byte slots per row
    const int k = q * (64 / S) + lane / S;
    const int slot = lane % S;
    const int i = i0 + (F32 ? slot * V : ((slot >> 1) ^ mn_key<R>(k)) * 16 + (slot & 1) * V);
    return Piece{k, i < end ? i : 0, k};
  };
  // piece x: A's (x < MI), then B's
  auto piece = [&](int x) {
    if (x < MI) {
      const int q = x * 4 + wave;
      if constexpr (K_::A_KC) return piece_kc(q, [&](int r) { return min(r, tl.rows - 1); });
      else return piece_mn(std::integral_constant<int, BM>{}, q, tl.m0, a.M);
    }
    const int q = (x - MI) * 4 + wave;
    if constexpr (K_::B_KC) return piece_kc(q, b_row);
    else return piece_mn(std::integral_constant<int, BN>{}, q, n0, a.N);
  };
  // byte offsets of the lane's pieces; 32 bits unless the operand's rows of one
  // k-step (an expert's whole weight if k-contiguous) reach over 4 GiB
  const bool narrow = max(a.lda * BM, a.ldb * (K_::B_KC ? max(BN, a.N) : BN)) <
                      (1L << 32) / (long)sizeof(T);
  unsigned off[MI + NJ];
#pragma unroll
  for (int x = 0; x < MI + NJ; ++x) {
    const Piece p = piece(x);
    off[x] = ((unsigned)p.r * (unsigned)(x < MI ? a.lda : a.ldb) + (unsigned)p.c) *
             (unsigned)sizeof(T);
  }
  const long a_step = K_::A_KC ? BK : BK * a.lda, b_step = K_::B_KC ? BK : BK * a.ldb;
  // the operands at the next k-step to load, and that k-step's first k
  const T *An = A, *Bn = B;
  int kn = 0;
  // piece x of the next k-step into stage st.  The last, partial k-step (and
  // every one where 32 bits do not reach) takes per-lane addresses, zeros past Kd.
  auto load = [&](char* st, int x) {
    char* dst = st + (x < MI ? x * 4 : A_BYTES / 1024 + (x - MI) * 4) * 1024 + wave * 1024;
    const T* base = x < MI ? An : Bn;
    if (narrow && kn + BK <= Kd) {
      dma16(base, off[x], dst);
    } else {
      const Piece p = piece(x);
      const T* src = base + (size_t)p.r * (x < MI ? a.lda : a.ldb) + p.c;
      dma16(kn + p.k < Kd ? (const void*)src : kZeros, dst);
    }
  };
  auto advance = [&]() {
    An += a_step;
    Bn += b_step;
    kn += BK;
  };

  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // fragment of an MFMA tile of k-block q: the 4 k (fp32) or 8 k (bf16) of a lane
  typedef typename std::conditional<F32, f32x4_t, bf16x8_t>::type Frag;
  auto frags = [&](auto kc, auto ntag, const char* op, int w, int q, Frag* f) {
    constexpr int N = decltype(ntag)::value;
    if constexpr (decltype(kc)::value) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int r = (w * N + i) * 16 + l16;
        f[i] = *reinterpret_cast<const Frag*>(op + r * 128 + (((4 * q + g4) ^ ((r >> 1) & 7)) << 4));
      }
    } else if constexpr (F32) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        typedef __attribute__((__vector_size__(N * 4))) float vN;
        const vN v = *reinterpret_cast<const vN*>(
            op + ((16 * q + 4 * g4 + e) * 32 * N + (w * 16 + l16) * N) * 4);
#pragma unroll
        for (int i = 0; i < N; ++i) f[i][e] = v[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        s16x4_t v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = 32 * q + 8 * g4 + 4 * h + (l16 >> 2);
          v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(
              op + k * (64 * N) + ((w * N + i) ^ mn_key<32 * N>(k)) * 32 + (l16 & 3) * 8));
        }
        f[i] = __builtin_bit_cast(Frag, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
      }
    }
  };

  // both operands' fragments of k-block q of a stage
  struct Frags {
    Frag a[MI], b[NJ];
  };
  auto read = [&](const char* st, int q, Frags& f) {
    frags(std::bool_constant<K_::A_KC>{}, std::integral_constant<int, MI>{}, st, wm, q, f.a);
    frags(std::bool_constant<K_::B_KC>{}, std::integral_constant<int, NJ>{}, st + A_BYTES, wn, q, f.b);
  };
  // the MFMAs of a k-block; between(e) is issued after the e-th quarter
  auto mma = [&](const Frags& f, auto&& between) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          if constexpr (F32)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.b[j][e], f.a[i][e], acc[i][j], 0, 0, 0);
          else if ((i * NJ + j) * 4 / (MI * NJ) == e)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
        }
      between(e);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int p = 0; p < NS; ++p)
    if (p < nk) {
#pragma unroll
      for (int x = 0; x < MI + NJ; ++x) load(lds + p * STAGE, x);
      advance();
    }
  // Each k-block's fragments are read while the previous block's MFMAs run.
  // Between the two blocks of k-step kt (its second fragments already in
  // registers) a wave waits for its pieces of k-step kt + 1 (later ones stay
  // in flight) and takes the barrier after which every wave's have landed and
  // stage kt is free: k-step kt + NS goes there, its pieces issued between the
  // MFMAs.  (Issued ahead of them, they and the barrier cost a lone wave of a
  // SIMD 530 clocks per k-step, as much as the MFMAs of a 32 x 64 tile.)
  Frags f0, f1;
  if (nk > 0) {
    wait_vm_groups<MI + NJ, NS - 1>(nk - 1);
    __syncthreads();
    read(lds, 0, f0);
  }
  char* st = lds;
  for (int kt = 0; kt < nk; ++kt) {
    read(st, 1, f1);
    char* const next = st == lds + (NS - 1) * STAGE ? lds : st + STAGE;
    __builtin_amdgcn_sched_barrier(0);
    mma(f0, [](int) {});
    WAIT_LGKMCNT(0);  // f1 (here, so that its use below waits for nothing read later)
    if (kt + 1 < nk) {
      wait_vm_groups<MI + NJ, NS - 2>(nk - 2 - kt);
      __syncthreads();
      read(next, 0, f0);
    }
    __builtin_amdgcn_sched_barrier(0);
    const bool refill = kt + NS < nk;
    mma(f1, [&](int e) {
      constexpr int PER = (MI + NJ + 3) / 4;
      if (refill) {
#pragma unroll
        for (int x = 0; x < PER; ++x)
          if (e * PER + x < MI + NJ) load(st, e * PER + x);
      }
    });
    advance();
    st = next;
  }

  // epilogue, bf16 rows: through a wave-private region of the ring, so that every
  // global access is 16 bytes of a row and 2 NJ (GU_FWD: NJ) lanes in a row
  // take consecutive ones.  (With the accumulators' own 8-byte pieces, GU of
  // 8192 rows, H = 1408 and a single k-step took 34 us against 24 in the large
  // tiles.)  Chunk c (16 bytes) of row r sits at chunk c ^ key(r).
  if constexpr (!F32 && K_::MRAG) {
    constexpr int CPR = 2 * NJ;  // chunks per row
    char* reg = lds + wave * (16 * MI * CPR * 16);
    auto at = [&](int r, int c) { return reg + (r * CPR + (c ^ ((r >> 1) & (CPR - 1)))) * 16; };
    __syncthreads();  // every wave is done with the ring
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        *reinterpret_cast<bf16x4_t*>(at(16 * i + l16, 2 * j + (g4 >> 1)) + (g4 & 1) * 8) =
            __builtin_convertvector(acc[i][j], bf16x4_t);
    const int rows = tl.rows - wm * 16 * MI;  // of this wave's
    if constexpr (KIND == GU_FWD) {
      constexpr int RPP = 64 / NJ;  // rows per pass
      const int c = lane % NJ, h = (n0 >> 1) + wn * 8 * NJ + 8 * c;
#pragma unroll
      for (int r0 = 0; r0 < 16 * MI; r0 += RPP) {
        const int r = r0 + lane / NJ;
        if (r >= 16 * MI || r >= rows || h >= a.H) continue;
        const bf16x8_t G = *reinterpret_cast<const bf16x8_t*>(at(r, c));
        const bf16x8_t U = *reinterpret_cast<const bf16x8_t*>(at(r, c + NJ));
        bf16x8_t Hv;
#pragma unroll
        for (int e = 0; e < 8; ++e) Hv[e] = (bf16_t)(silu_t<T>((float)G[e]) * (float)U[e]);
        const size_t m = (size_t)(tl.row0 + wm * 16 * MI + r);
        put8(a.C, m * 2 * a.H + h, G);
        put8(a.C, m * 2 * a.H + a.H + h, U);
        put8(a.out2, m * a.H + h, Hv);
      }
    } else {
      constexpr int RPP = 64 / CPR, P = (16 * MI + RPP - 1) / RPP;
      const int c = lane % CPR, n = n0 + wn * 16 * NJ + 8 * c;
      const bool ok = n < a.N;
      // (dSwiGLU, dSiLU) the stored G, U or A of all rows, before the first use
      bf16x8_t G[P], U[P];
      if constexpr (KIND == DHH_BWD || KIND == DH_BWD) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const int r = p * RPP + lane / CPR;
          const size_t m = (size_t)(tl.row0 + wm * 16 * MI + r);
          if (!ok || r >= rows) continue;
          if constexpr (KIND == DHH_BWD) {
            G[p] = get8(a.aux, m * 2 * a.H + n);
            U[p] = get8(a.aux, m * 2 * a.H + a.H + n);
          } else {
            G[p] = get8(a.aux, m * a.H + n);
          }
        }
      }
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int r = p * RPP + lane / CPR;
        const size_t m = (size_t)(tl.row0 + wm * 16 * MI + r);
        if (!ok || r >= 16 * MI || r >= rows) continue;
        bf16x8_t v = *reinterpret_cast<const bf16x8_t*>(at(r, c));
        if constexpr (KIND == DHH_BWD) {
          // dG = dHh U silu'(G), dU = dHh silu(G)
          bf16x8_t dG, dU;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float g = (float)G[p][e], dh = (float)v[e];
            dG[e] = (bf16_t)(dh * (float)U[p][e] * dsilu_t<T>(g));
            dU[e] = (bf16_t)(dh * silu_t<T>(g));
          }
          put8(a.C, m * 2 * a.H + n, dG);
          put8(a.C, m * 2 * a.H + a.H + n, dU);
        } else if constexpr (KIND == DH_BWD) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = (bf16_t)((float)v[e] * dsilu_t<T>((float)G[p][e]));
          put8(a.C, m * a.ldc + n, v);
        } else {
          put8(a.C, m * a.ldc + n, v);
          if constexpr (KIND == UP_FWD) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (bf16_t)silu_t<T>((float)v[e]);
            put8(a.out2, m * a.H + n, v);
          }
        }
      }
    }
  } else {
    // epilogue, straight from the accumulators
    const int m_end = K_::MRAG ? tl.rows : a.M - tl.m0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      // (fp32 m/n-contiguous operands: a lane's MI indices are consecutive)
      const int r = K_::A_KC || !F32 ? (wm * MI + i) * 16 + l16 : (wm * 16 + l16) * MI + i;
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
          for (int e = 0; e < 4; ++e) Hv[e] = silu_t<float>(G[e]) * U[e];
          put4(a.C, m * 2 * a.H + h, G);
          put4(a.C, m * 2 * a.H + a.H + h, U);
          put4(a.out2, m * a.H + h, Hv);
        }
      } else {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          int n;
          f32x4_t v;
          if constexpr (K_::B_KC || !F32) {
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
}

constexpr int kXcds = 8;
constexpr int kBand = 8;  // m-tiles per band of the tile order

template <int KIND>
DEVI constexpr int cols_of(const GemmArgs& a) { return KIND == GU_FWD ? 2 * a.H : a.N; }

// Weight gradients (ragged in K): a group's tiles all take its own number of
// k-steps, so of uneven groups every XCD takes an eighth of each one's per_group
// tiles, XCD x the ((x + g) % 8)-th of group g (eighths that differ by a tile then
// even out).  With an eighth of all tiles, the XCDs that got a large group worked
// on alone.  Zipf-sized groups, fp32: 1531 rows in 6, d = 520, H = 1408, forward
// and backward 327 -> 264 us; 4096 rows in 8, d = 1024, the same H, backward 1190 ->
// 619; bf16, 3000 rows in 24, d = 960, H = 512 73 -> 64.  Even groups keep an eighth
// of all (fewer XCDs read the same rows: 1500 rows in 12, d = 768, H = 704: 51 -> 49 us).
constexpr int kTileRows = 128;  // a tile's fill and epilogue, in rows of its reduction
DEVI int eighth(int per_group, int x) { return (int)((long)per_group * x / kXcds); }

// Tile order: XCD x takes the x-th eighth of every set's tiles (blocks go to the XCDs
// round-robin by id), in bands of kBand m-tiles, or an eighth of every uneven group's.
// The grid covers the largest number of tiles that the group sizes can give; blocks
// past the last tile end at once.
template <class T, int KA, int KB, int MI, int NJ, int NS>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(GemmLaunch L) {
  constexpr int BM = 32 * MI, BN = 32 * NJ;
  constexpr int RING = NS * (BM + BN) * 128;
  static_assert(RING >= (int)sizeof(GroupTable) * (KA == KB ? 2 : 4), "the group tables share the ring");
  __shared__ __attribute__((aligned(1024))) char lds[RING];
  GroupTable* gtab = reinterpret_cast<GroupTable*>(lds);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wave < L.n_sets) build_group_table<BM>(L.s[wave], gtab[wave], kTileRows);
  __syncthreads();
  const int xcd = blockIdx.x % kXcds;
  int i = blockIdx.x / kXcds;  // this block's tile among the XCD's
  int set = -1;
  TileAt tl{};
  for (int q = 0; q < L.n_sets; ++q) {
    const GemmArgs& a = L.s[q];
    const bool kb = KA != KB && L.kind_b[q] != 0;
    const bool mrag = kb ? Kind<KB>::MRAG : Kind<KA>::MRAG;
    const int cols = kb ? cols_of<KB>(a) : cols_of<KA>(a);
    const int mt_g = mrag ? 0 : (a.M + BM - 1) / BM;
    const int n_tiles = (cols + BN - 1) / BN;
    if (!mrag && __builtin_amdgcn_readfirstlane(gtab[q].uneven)) {
      const int per_group = mt_g * n_tiles;
      auto share = [&](int g) {
        const int y = (xcd + g) % kXcds;
        return eighth(per_group, y + 1) - eighth(per_group, y);
      };
      int cnt = a.n_groups / kXcds * per_group;
      for (int g = a.n_groups / kXcds * kXcds; g < a.n_groups; ++g) cnt += share(g);
      if (i >= cnt) {
        i -= cnt;
        continue;
      }
      set = q;
      // eight groups in a row make per_group tiles
      int g = i / per_group * kXcds;
      i %= per_group;
      for (; i >= share(g); ++g) i -= share(g);
      int r = eighth(per_group, (xcd + g) % kXcds) + i;
      const int first_m = r / (kBand * n_tiles) * kBand;
      const int band_m = min(kBand, mt_g - first_m);
      r -= first_m * n_tiles;
      tl.tile_n = r / band_m;
      tl.g = g;
      tl.m0 = (first_m + r % band_m) * BM;
      tl.row0 = gtab[q].c[g];
      tl.rows = max(0, gtab[q].c[g + 1] - tl.row0);
      break;
    }
    const int m_tiles = __builtin_amdgcn_readfirstlane(mrag ? gtab[q].p[a.n_groups] : a.n_groups * mt_g);
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
      gemm_tile<T, KB, MI, NJ, NS>(L.s[set], tl, lds);
      return;
    }
  }
  gemm_tile<T, KA, MI, NJ, NS>(L.s[set], tl, lds);
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

template <class T, int KA, int KB, int MI, int NJ, int NS>
hipError_t launch(const GemmArgs* sa, int na, const GemmArgs* sb, int nb, hipStream_t s) {
  GemmLaunch L{};
  long blocks = 0;
  auto add = [&](const GemmArgs& a, int kb, long tiles) {
    L.s[L.n_sets] = a;
    L.kind_b[L.n_sets++] = kb;
    long per_xcd = (tiles + kXcds - 1) / kXcds;
    if (!(kb ? Kind<KB>::MRAG : Kind<KA>::MRAG) && a.n_groups > 0) {
      // every eight groups deal an XCD per_group tiles, the last few at most an
      // eighth of theirs, rounded up
      const long per_group = tiles / a.n_groups, rest = a.n_groups % kXcds;
      per_xcd = a.n_groups / kXcds * per_group +
                std::min(per_group, rest * ((per_group + kXcds - 1) / kXcds));
    }
    blocks += kXcds * per_xcd;
  };
  // longest reduction per tile first (K-ragged kinds: the mean group's rows), so
  // that no long tile starts last
  struct Entry {
    const GemmArgs* a;
    int kb;
    long k, tiles;
  } e[kMaxSets];
  int n = 0;
  auto len = [](bool mrag, const GemmArgs& a) {
    return mrag ? (long)a.K : (long)a.cap / std::max(1, a.n_groups);
  };
  for (int q = 0; q < na; ++q)
    e[n++] = Entry{&sa[q], 0, len(Kind<KA>::MRAG, sa[q]), max_tiles<KA, MI, NJ>(sa[q])};
  for (int q = 0; q < nb; ++q)
    e[n++] = Entry{&sb[q], 1, len(Kind<KB>::MRAG, sb[q]), max_tiles<KB, MI, NJ>(sb[q])};
  std::stable_sort(e, e + n, [](const Entry& x, const Entry& y) { return x.k > y.k; });
  for (int q = 0; q < n; ++q) add(*e[q].a, e[q].kb, e[q].tiles);
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffffL) return hipErrorInvalidConfiguration;
  MOE_TIMED((kTileNames[gemm_name_index(KA, KB)]), s,
            gemm_tile_kernel<T, KA, KB, MI, NJ, NS><<<(unsigned)blocks, 256, 0, s>>>(L));
  return hipGetLastError();
}

template <class T, int KA, int KB>
hipError_t run_kinds(const GemmArgs* sa, int na, const GemmArgs* sb, int nb, TileSize size,
                     hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    if constexpr (KA == KB) {
      if (size == TILE_32x64) return launch<T, KA, KB, 1, 2, 6>(sa, na, sb, nb, s);
    }
    if (size == TILE_64x64) return launch<T, KA, KB, 2, 2, 3>(sa, na, sb, nb, s);
    return launch<T, KA, KB, 2, 4, 2>(sa, na, sb, nb, s);
  } else {
    // Six tiles of 64 x 128 per CU (by the bound on the group sizes) keep every
    // SIMD busy and halve the L2 traffic; with fewer, 32 x 64 tiles fill the CUs
    // and pad ragged groups less.  Measured (us, 64 x 128 / 32 x 64): 4096 rows,
    // d = 1024, H = 1408, 8 groups: GU (1584 tiles) 210 / 227, dX + dW_gu (3392)
    // 401 / 447, down projection (576) 138 / 122; 1531 rows, d = 520, 6 groups:
    // GU (660) 65 / 59, down projection (150) 60 / 36.  Tiles of 64 x 64 and
    // 128 x 128 were no better than these two in any of them.
    if (launch_tiles<KA, KB, 2, 4>(sa, na, sb, nb) >= 6L * num_cus())
      return launch<T, KA, KB, 2, 4, 2>(sa, na, sb, nb, s);
    return launch<T, KA, KB, 1, 2, 3>(sa, na, sb, nb, s);
  }
}

}  // namespace

hipError_t run_gemm_tile(int bf16, int ka, int kb, const GemmArgs* sa, int na, const GemmArgs* sb,
                         int nb, TileSize size, hipStream_t s) {
#define MOE_KINDS(A, B)                                                          \
  if (ka == A && kb == B)                                                        \
    return bf16 ? run_kinds<bf16_t, A, B>(sa, na, sb, nb, size, s)                 \
              : run_kinds<float, A, B>(sa, na, sb, nb, size, s)
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
