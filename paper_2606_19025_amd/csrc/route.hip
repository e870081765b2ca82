// Router: logits over all E experts, top-k, gate weights, ghost-expert mask,
// and the router backward.
//
// Forward (App. A: TopK of the router scores; Sec. 3.3: the router stays
// unpartitioned under skip-token, routes to non-resident experts are masked):
//   one block = 32 tokens, 8 waves.  bf16 logits use v_mfma_f32_32x32x16_bf16
//   (tokens x experts tiles, the d reduction split over the 8 waves and summed
//   in a fixed order through LDS; x and, for up to 64 experts, W_r rows are
//   read whole and staged in LDS); for more experts the waves split the
//   experts (logits_ring).  fp32 layers run one v_mfma_f32_16x16x4_f32 chain
//   per logit (logits_f32).  For
//   k <= 8 every wave then selects for 4 tokens, 16 lanes per token
//   (select_groups, row maxima by DPP); for larger k each wave takes tokens
//   one at a time, lane = expert, with k wave-wide (max logit, min id)
//   reductions.
#include "common.h"
#include "kernels.h"
#include "timing.h"

namespace moe {
namespace {

constexpr int RT_TOK = 32;   // tokens per block
constexpr int RT_WAVES = 8;
constexpr int RT_THREADS = 64 * RT_WAVES;

struct RouteFwdArgs {
  const void* x;
  const void* w;
  const float* bias;
  const uint8_t* resident;
  float* logits;
  int32_t* idx;
  float* tw;
  int32_t* local;
  int T, d, E, k, gate;
  float inv_tau;
};

// Wave-wide (value desc, id asc) argmax.
DEVI void wave_argmax(float& v, int& e) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(v, o, 64);
    int oe = __shfl_xor(e, o, 64);
    if (ov > v || (ov == v && oe < e)) { v = ov; e = oe; }
  }
}

// Local id (rank among resident experts, -1 for ghosts) of every expert, via
// ballots over chunks of 64 experts.  Executed by wave 0.
DEVI void build_local_map(const uint8_t* resident, int E, int* lmap) {
  const int lane = threadIdx.x & 63;
  int base = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int e = e0 + lane;
    const bool r = (e < E) && resident[e] != 0;
    const uint64_t m = __ballot(r);
    const int below = __popcll(m & ((1ull << lane) - 1ull));
    if (e < E) lmap[e] = r ? base + below : -1;
    base += __popcll(m);
  }
}

// z = (sum of the P partial dot products, in order, + bias) * inv_tau of the
// block's tokens, from part [P][RT_TOK][EP], into zl[RT_TOK][ldz] and the
// caller's logits.
template <int EP, int P>
DEVI void finish_logits(const RouteFwdArgs& a, int t0, const float* part, float* zl, int ldz) {
  for (int p = threadIdx.x; p < RT_TOK * EP; p += RT_THREADS) {
    const int i = p / EP, e = p % EP;
    float v = part[p];
#pragma unroll
    for (int q = 1; q < P; ++q) v += part[q * (RT_TOK * EP) + p];
    if (e < a.E) {
      if (a.bias) v += a.bias[e];
      v *= a.inv_tau;
      zl[i * ldz + e] = v;
      const int t = t0 + i;
      if (a.logits && t < a.T) a.logits[(size_t)t * a.E + e] = v;
    }
  }
  __syncthreads();
}

// bf16 logits of RT_TOK tokens into zl[RT_TOK][ldz], for up to 64 experts and
// d past what logits_mfma_staged takes.
// Wave w reduces the 64-wide slices w, w + RT_WAVES, ... of d, up to two
// slices per round with all their loads issued before the MFMAs; the per-wave partial
// sums are then added in wave order through LDS.
template <int NEB>
DEVI void logits_mfma(const RouteFwdArgs& a, int t0, float* zl, int ldz) {
  const bf16_t* x = static_cast<const bf16_t*>(a.x);
  const bf16_t* w = static_cast<const bf16_t*>(a.w);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int row = lane & 31;
  const int half = lane >> 5;
  f32x16_t acc[NEB];
#pragma unroll
  for (int eb = 0; eb < NEB; ++eb) acc[eb] = f32x16_t{};
  const bf16x8_t zero8 = {};
  const u32x4_t zero4 = {0u, 0u, 0u, 0u};
  const int n_slices = (a.d + 63) / 64;
  // x slices go through a wave-private LDS buffer: loaded as whole 128-byte
  // row pieces (8 lanes per token row; 32 rows per read in fragment order
  // would touch 32 cache lines per instruction), stored with the 16-byte
  // chunk c of row r at chunk position c ^ ((r >> 1) & 7) so that the
  // fragment reads (16 consecutive rows, same chunk) are free of bank
  // conflicts.  The W slices stay direct fragment loads (L2-resident).
  static_assert(NEB <= 2, "up to 64 experts");
  constexpr int UNR = 2;
  __shared__ __attribute__((aligned(16))) char xst[RT_WAVES][UNR][RT_TOK * 128];
  auto xswz = [](int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); };
  auto load_x = [&](int kb, u32x4_t* v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int tr = t0 + j * 8 + (lane >> 3);
      const int c = kb * 64 + (lane & 7) * 8;
      v[j] = (kb < n_slices && tr < a.T && c + 8 <= a.d)
                 ? *reinterpret_cast<const u32x4_t*>(x + (size_t)tr * a.d + c)
                 : zero4;
    }
  };
  auto store_x = [&](int u, const u32x4_t* v) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<u32x4_t*>(&xst[wave][u][xswz(j * 8 + (lane >> 3), lane & 7)]) = v[j];
  };
  // the lane's 32 consecutive elements of a slice feed the 4 k16 MFMA steps
  // in the same order for the token and the expert operand
  auto read_x = [&](bf16x8_t* av, int u) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      av[q] = *reinterpret_cast<const bf16x8_t*>(&xst[wave][u][xswz(row, half * 4 + q)]);
  };
  auto load_w = [&](int kb, bf16x8_t (*bv)[4]) {
    const int c0 = kb * 64 + half * 32;
#pragma unroll
    for (int eb = 0; eb < NEB; ++eb) {
      const int e = eb * 32 + row;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = c0 + q * 8;
        bv[eb][q] = (kb < n_slices && e < a.E && c + 8 <= a.d)
                        ? *reinterpret_cast<const bf16x8_t*>(w + (size_t)e * a.d + c) : zero8;
      }
    }
  };
  // UNR slices per round (fewer for wide expert sets, to stay in registers)
  for (int kb = wave; kb < n_slices; kb += UNR * RT_WAVES) {
    bf16x8_t av[UNR][4], bv[UNR][NEB][4];
    u32x4_t xv[UNR][4];
    // the W_r fragments (L2) are requested with the x rows (HBM), not after
    // the x rows have been staged
#pragma unroll
    for (int u = 0; u < UNR; ++u) load_w(kb + u * RT_WAVES, bv[u]);
#pragma unroll
    for (int u = 0; u < UNR; ++u) load_x(kb + u * RT_WAVES, xv[u]);  // zeros past the end
#pragma unroll
    for (int u = 0; u < UNR; ++u) store_x(u, xv[u]);
#pragma unroll
    for (int u = 0; u < UNR; ++u) read_x(av[u], u);
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[u][q], bv[u][eb][q], acc[eb], 0, 0, 0);
  }
  // deterministic cross-wave sum (wave order): every wave stores its partial
  // tile, then each thread adds its entries' RT_WAVES partials and finishes z
  // (bias, temperature, logits store)
  __shared__ float part[RT_WAVES][RT_TOK * NEB * 32];
#pragma unroll
  for (int eb = 0; eb < NEB; ++eb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = (r >> 2) * 8 + half * 4 + (r & 3);
      part[wave][i * NEB * 32 + eb * 32 + row] = acc[eb][r];
    }
  }
  __syncthreads();
  finish_logits<NEB * 32, RT_WAVES>(a, t0, &part[0][0], zl, ldz);
}

// bf16 logits for up to 64 experts and d <= 64 XS RT_WAVES.  Wave w reduces
// the slices w + RT_WAVES u (u < XS) of d.  The x rows and W_r rows of a
// slice are read whole (8 lanes per 128-byte row piece, two slices ahead of
// their use, into registers) and staged in the wave's own LDS region, from
// which the MFMA fragments are read.  (Read in fragment order instead, 32
// rows per load, W_r took twice as long to arrive.)  The per-wave partial
// sums are then added in wave order through LDS and z is finished as in
// logits_mfma.
template <int NEB, int XS>
DEVI void logits_mfma_staged(const RouteFwdArgs& a, int t0, float* zl, int ldz) {
  static_assert(NEB <= 2 && XS >= 2, "up to 64 experts, at least two slices per wave");
  const bf16_t* x = static_cast<const bf16_t*>(a.x);
  const bf16_t* w = static_cast<const bf16_t*>(a.w);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int row = lane & 31;
  const int half = lane >> 5;
  constexpr int XR = RT_TOK, WR = NEB * 32;  // x and W_r rows of a slice
  constexpr int SLOT = (XR + WR) * 128;
  constexpr int STG = RT_WAVES * SLOT;
  constexpr int PART = RT_WAVES * RT_TOK * NEB * 32 * 4;
  __shared__ __attribute__((aligned(16))) char lbuf[STG > PART ? STG : PART];
  char* slot = lbuf + wave * SLOT;
  // 16-byte chunk c of staged row r at chunk position c ^ ((r >> 1) & 7): the
  // fragment reads (16 consecutive rows, one chunk) are free of bank conflicts
  auto swz = [](int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); };
  const int n_slices = (a.d + 63) / 64;
  const u32x4_t zero4 = {0u, 0u, 0u, 0u};
  struct Piece {
    u32x4_t x[XR / 8], w[WR / 8];
  };
  auto load = [&](int kb, Piece& p) {
    const int c = kb * 64 + (lane & 7) * 8;
    const bool ok = kb < n_slices && c + 8 <= a.d;
#pragma unroll
    for (int j = 0; j < XR / 8; ++j) {
      const int t = t0 + j * 8 + (lane >> 3);
      p.x[j] = ok && t < a.T ? *reinterpret_cast<const u32x4_t*>(x + (size_t)t * a.d + c) : zero4;
    }
#pragma unroll
    for (int j = 0; j < WR / 8; ++j) {
      const int e = j * 8 + (lane >> 3);
      p.w[j] = ok && e < a.E ? *reinterpret_cast<const u32x4_t*>(w + (size_t)e * a.d + c) : zero4;
    }
  };
  f32x16_t acc[NEB];
#pragma unroll
  for (int eb = 0; eb < NEB; ++eb) acc[eb] = f32x16_t{};
  Piece pc[XS];
  load(wave, pc[0]);
  load(wave + RT_WAVES, pc[1]);
#pragma unroll
  for (int u = 0; u < XS; ++u) {
    const int kb = wave + u * RT_WAVES;
    if (kb >= n_slices) break;
    // a wave's LDS accesses run in order: the previous slice's fragment
    // reads are done before these stores overwrite them
#pragma unroll
    for (int j = 0; j < XR / 8; ++j)
      *reinterpret_cast<u32x4_t*>(slot + swz(j * 8 + (lane >> 3), lane & 7)) = pc[u].x[j];
#pragma unroll
    for (int j = 0; j < WR / 8; ++j)
      *reinterpret_cast<u32x4_t*>(slot + XR * 128 + swz(j * 8 + (lane >> 3), lane & 7)) = pc[u].w[j];
    if (u + 2 < XS) load(kb + 2 * RT_WAVES, pc[u + 2]);
    bf16x8_t av[4], bv[NEB][4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      av[q] = *reinterpret_cast<const bf16x8_t*>(slot + swz(row, half * 4 + q));
#pragma unroll
    for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        bv[eb][q] = *reinterpret_cast<const bf16x8_t*>(slot + XR * 128 + swz(eb * 32 + row, half * 4 + q));
#pragma unroll
    for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[q], bv[eb][q], acc[eb], 0, 0, 0);
  }
  __syncthreads();  // every wave is done with its staging region: the partial sums reuse it
  float* part = reinterpret_cast<float*>(lbuf);
#pragma unroll
  for (int eb = 0; eb < NEB; ++eb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = (r >> 2) * 8 + half * 4 + (r & 3);
      part[wave * (RT_TOK * NEB * 32) + i * NEB * 32 + eb * 32 + row] = acc[eb][r];
    }
  }
  __syncthreads();
  finish_logits<NEB * 32, RT_WAVES>(a, t0, part, zl, ldz);
}

// Address of zeros for k past the last (16 bytes).
__device__ __attribute__((aligned(16))) const uint32_t kRouteZeros[4] = {0u, 0u, 0u, 0u};

// 16 (or 4) bytes per lane at p -> LDS at base + 16 (4) lane, base wave-uniform.
// The asm sets m0 and leaves the one wait state an LDS DMA needs after it.
template <bool VEC>
DEVI void route_dma(const void* p, char* base) {
  const unsigned m0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_t*)base);
  if constexpr (VEC)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(m0)
                 : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(p), "s"(m0)
                 : "m0", "memory");
}

// bf16 logits of more than 64 experts.  The waves form EG expert groups (32
// experts each) x KG = 8 / EG groups of d slices: a wave's 32 x 32 tile of
// (token, expert) runs over the slices kg, kg + KG, ... of 64, so W_r is read
// once per block, each row by one wave.  (One wave for all experts of a d slice
// held 128 accumulators at 256 experts and added them to LDS wave after wave:
// 5003 tokens, d = 1536, 256 experts took 82 us, now 26, bound by each CU's read of
// W_r (786 KB) from L2.)
// The sums are those of the narrower paths, to the bit: slices s, s + 8, ... in
// one accumulator, the same 16 of d in each MFMA, and the eight accumulators
// added in order, so that a logit does not depend on how many experts there are
// (a rounding's difference is enough to swap two ranks).
// x and W_r rows go to LDS by DMA as whole 128-byte pieces through a ring of NS
// stages.  Chunk c (16 bytes) of row r sits at chunk c ^ ((r >> 1) & 7).
template <int EG>
DEVI void logits_ring(const RouteFwdArgs& a, int t0, float* zl, int ldz) {
  constexpr int KG = RT_WAVES / EG;
  constexpr int EP = EG * 32;
  constexpr int KW = 64;                          // elements of a slice
  constexpr int W_BYTES = RT_WAVES * 4096;        // each wave's 32 W_r rows
  constexpr int STAGE = W_BYTES + KG * 4096;      // and the KG slices' 32 x rows
  constexpr int NS = 3;
  constexpr int XP = KG >= 2 ? KG / 2 : 1;        // KiB of x per wave and stage
  constexpr int PER = 4 + XP;                     // DMA loads per wave and stage
  constexpr int NA = RT_WAVES / KG;               // a wave's share of the 8 sums
  constexpr int P = KG == 1 ? 1 : RT_WAVES;       // sums left to add through LDS
  constexpr int PART = P * RT_TOK * EP * 4;
  __shared__ __attribute__((aligned(1024))) char ring[NS * STAGE > PART ? NS * STAGE : PART];
  const bf16_t* x = static_cast<const bf16_t*>(a.x);
  const bf16_t* w = static_cast<const bf16_t*>(a.w);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int eg = wave % EG, kg = wave / EG;
  const int n_slices = (a.d + KW - 1) / KW;
  const int n_stages = (n_slices + KG - 1) / KG;
  // one KiB (8 rows of 128 bytes, from row r0) of slice sl of p into dst; row
  // index clamped to the last (the results of the rows past it are not used)
  auto kib = [&](const bf16_t* p, int r0, int last, int sl, char* dst) {
    const int r = r0 + (lane >> 3);
    const int c = ((lane & 7) ^ ((r >> 1) & 7)) * 8 + sl * KW;
    route_dma<true>(c < a.d ? (const void*)(p + (size_t)min(r, last) * a.d + c) : kRouteZeros, dst);
  };
  auto load = [&](int stage) {
    char* st = ring + stage % NS * STAGE;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      kib(w, eg * 32 + 8 * i, a.E - 1, stage * KG + kg, st + wave * 4096 + i * 1024);
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      // the block's 4 KG KiB of x (EG = 8: waves w and w + 4 bring the same one)
      const int q = (wave * XP + i) % (4 * KG);
      kib(x, t0 + 8 * (q & 3), a.T - 1, stage * KG + (q >> 2), st + W_BYTES + q * 1024);
    }
  };
  f32x16_t acc[NA];
#pragma unroll
  for (int u = 0; u < NA; ++u) acc[u] = f32x16_t{};
  const int row = lane & 31, half = lane >> 5;
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < n_stages) load(p);
  for (int s0 = 0; s0 < n_stages; s0 += NA) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int s = s0 + u;
      if (s >= n_stages) break;
      wait_vm_groups<PER, NS - 2>(n_stages - 1 - s);
      __syncthreads();  // stage s is whole; everyone is done with stage s - 1
      if (s + NS - 1 < n_stages) load(s + NS - 1);
      const char* wl = ring + s % NS * STAGE + wave * 4096;
      const char* xl = ring + s % NS * STAGE + W_BYTES + kg * 4096;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int o = row * 128 + (((4 * half + q) ^ ((row >> 1) & 7)) << 4);
        acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(xl + o),
                                                         *reinterpret_cast<const bf16x8_t*>(wl + o),
                                                         acc[u], 0, 0, 0);
      }
    }
  }
  __syncthreads();  // the sums take the ring's place
  float* part = reinterpret_cast<float*>(ring);
  if constexpr (P == 1) {
#pragma unroll
    for (int u = 1; u < NA; ++u) acc[0] += acc[u];
  }
#pragma unroll
  for (int u = 0; u < (P == 1 ? 1 : NA); ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = (r >> 2) * 8 + half * 4 + (r & 3);
      part[((u * KG + kg) * RT_TOK + i) * EP + eg * 32 + row] = acc[u][r];
    }
  __syncthreads();
  finish_logits<EP, P>(a, t0, part, zl, ldz);
}

// fp32 logits.  A logit is one chain of fused multiply-adds in the order of d,
// the order that a plain loop takes: v_mfma_f32_16x16x4_f32 adds its four products
// one after another, each rounded once, so a chain of them gives the loop's bits.
// (Ranks hang on these bits: with d split over waves and four accumulators, two
// logits of a token within rounding of each other came out in the other order in
// one of some 150 calls, and with them whole rows of the gradients.)
// A block's tiles of 16 tokens x 16 experts are shared out over the waves, so that
// all four SIMDs issue MFMAs from 32 experts on: 8192 tokens, d = 2048, 64 experts
// 36 us (32 with d split; 1913 with a thread's loop per logit), 5003 tokens, d =
// 1536, 256 experts 83 (78; 5882), 256 tokens, d = 64, 8 experts 6.4 (7.1; 9.7).
// x and W_r rows come to LDS by DMA as whole 128-byte pieces (a slice, 32 of d)
// through a ring of NS stages of KS slices.  Chunk c (16 bytes) of row r sits at
// chunk c ^ ((r >> 1) & 7).  VEC: rows are 16-byte aligned; otherwise the DMA
// moves 4 bytes per lane.
template <int EP, bool VEC>
DEVI void logits_f32(const RouteFwdArgs& a, int t0, float* zl, int ldz) {
  constexpr int KW = 32;                                // elements of a slice
  constexpr int KS = EP == 256 ? 1 : EP == 128 ? 2 : 4;  // slices of a stage
  constexpr int NS = 3;
  constexpr int ROWS = RT_TOK + EP;                     // x rows, then W_r rows
  constexpr int SLICE = ROWS * 128, STAGE = KS * SLICE;
  constexpr int PIECES = STAGE / 1024;                  // of 8 rows
  constexpr int PER_WAVE = (PIECES + RT_WAVES - 1) / RT_WAVES;
  constexpr int PER = PER_WAVE * (VEC ? 1 : 4);         // DMA loads per wave and stage
  constexpr int MT = EP >= 128 ? 2 : 1;                 // a wave's tiles of 16 tokens
  constexpr int NT = EP == 256 ? 2 : 1;                 // and of 16 experts
  __shared__ __attribute__((aligned(1024))) char ring[NS * STAGE];
  const float* x = static_cast<const float*>(a.x);
  const float* w = static_cast<const float*>(a.w);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_stages = (a.d + KW * KS - 1) / (KW * KS);
  // rows past the last token or expert repeat it (their results are not used)
  auto row_at = [&](int r) {
    return r < RT_TOK ? x + (size_t)min(t0 + r, a.T - 1) * a.d
                      : w + (size_t)min(r - RT_TOK, a.E - 1) * a.d;
  };
  auto load = [&](int stage) {
    char* st = ring + stage % NS * STAGE;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      // (the last waves of a stage that does not divide bring its first pieces again)
      const int q = (wave * PER_WAVE + i) % PIECES;
      const int r0 = q % (ROWS / 8) * 8;
      const int k0 = (stage * KS + q / (ROWS / 8)) * KW;
      char* dst = st + q * 1024;
      if constexpr (VEC) {
        const int r = r0 + (lane >> 3);
        const int c = k0 + ((lane & 7) ^ ((r >> 1) & 7)) * 4;
        route_dma<true>(c < a.d ? (const void*)(row_at(r) + c) : kRouteZeros, dst);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = r0 + 2 * u + (lane >> 5);
          const int c = k0 + (((lane >> 2) & 7) ^ ((r >> 1) & 7)) * 4 + (lane & 3);
          route_dma<false>(c < a.d ? (const void*)(row_at(r) + c) : kRouteZeros, dst + u * 256);
        }
      }
    }
  };
  const int l16 = lane & 15, g4 = lane >> 4;
  const int tok0 = MT == 2 ? 0 : (wave & 1) * 16;
  const int exp0 = EP == 256 ? wave * 32 : EP == 128 ? wave * 16 : (wave >> 1) * 16;
  const bool busy = exp0 < EP && exp0 < a.E;
  // byte offset of element 4 m + g4 of a slice in row l16 of a 16-row tile
  int off[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) off[m] = l16 * 128 + ((m ^ ((l16 >> 1) & 7)) << 4) + g4 * 4;
  f32x4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < n_stages) load(p);
  for (int s = 0; s < n_stages; ++s) {
    wait_vm_groups<PER, NS - 2>(n_stages - 1 - s);
    __syncthreads();  // stage s is whole; everyone is done with stage s - 1
    if (s + NS - 1 < n_stages) load(s + NS - 1);
    if (!busy) continue;
    const char* xl = ring + s % NS * STAGE + tok0 * 128;
    const char* wl = ring + s % NS * STAGE + (RT_TOK + exp0) * 128;
#pragma unroll
    for (int q = 0; q < KS; ++q)
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        float xv[MT], wv[NT];
#pragma unroll
        for (int i = 0; i < MT; ++i)
          xv[i] = *reinterpret_cast<const float*>(xl + q * SLICE + i * 2048 + off[m]);
#pragma unroll
        for (int j = 0; j < NT; ++j)
          wv[j] = *reinterpret_cast<const float*>(wl + q * SLICE + j * 2048 + off[m]);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[i], wv[j], acc[i][j], 0, 0, 0);
      }
  }
  if (busy) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int e = exp0 + 16 * j + l16;
      if (e >= a.E) continue;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = tok0 + 16 * i + 4 * g4 + r;
          float v = acc[i][j][r];
          if (a.bias) v += a.bias[e];
          v *= a.inv_tau;
          zl[row * ldz + e] = v;
          if (a.logits && t0 + row < a.T) a.logits[(size_t)(t0 + row) * a.E + e] = v;
        }
    }
  }
  __syncthreads();
}

// Logit as read for selection: NaN ranks as -inf (some expert is always
// picked) and -0 as +0 (they tie, as equal values do).
DEVI float sel_value(float v) { return (v != v) ? -INFINITY : v + 0.0f; }

// Order-preserving map of a float to uint32 (larger float -> larger key);
// every float maps above 0, the key of an empty slot.
DEVI uint32_t sel_key(float v) {
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int RT_KSEL = 8;

// Lane permutations within a row of 16 lanes (DPP), applied to a 64-bit value
// (its two halves moved alike): xor 1 and xor 2 inside each quad, then lane
// i <- 7 - i inside each half-row and lane i <- 15 - i inside the row.  After
// taking the maximum with each in turn, every lane of the row holds the row's
// maximum.
template <int CTRL>
DEVI uint64_t row_perm64(uint64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, false);
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}
DEVI uint64_t max64(uint64_t a, uint64_t b) { return a > b ? a : b; }
DEVI uint64_t row16_max64(uint64_t m) {
  m = max64(m, row_perm64<0xB1>(m));   // quad_perm [1, 0, 3, 2]
  m = max64(m, row_perm64<0x4E>(m));   // quad_perm [2, 3, 0, 1]
  m = max64(m, row_perm64<0x141>(m));  // row_half_mirror
  m = max64(m, row_perm64<0x140>(m));  // row_mirror
  return m;
}

// Top-k (k <= RT_KSEL), gate weights and local ids of the block's tokens, 16
// lanes per token (all RT_WAVES waves: wave w takes tokens 4w .. 4w+3): lane
// s of a group holds experts s, s + 16, ... as 64-bit keys (order-preserving
// logit key, then the inverted expert id, so that equal logits rank the lower
// id first; 0 = taken or absent).  Round j takes the group's largest key (a
// row of 16 lanes, by DPP moves) and lane j keeps it, so the selections come
// out in rank order.
template <int LDZ, int NE>
DEVI void select_groups(const RouteFwdArgs& a, const float* zl, int t0, const int* lmap) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int s = lane & 15;
  const int i = wave * 4 + (lane >> 4);
  const int t = t0 + i;
  const float* z = zl + i * LDZ;
  uint64_t cand[NE];
#pragma unroll
  for (int q = 0; q < NE; ++q) {
    const int e = q * 16 + s;
    cand[q] = e < a.E ? ((uint64_t)sel_key(sel_value(z[e])) << 32) | (uint32_t)~e : 0ull;
  }
  int my_id = 0;
  for (int j = 0; j < a.k; ++j) {
    uint64_t m = 0ull;
#pragma unroll
    for (int q = 0; q < NE; ++q) m = cand[q] > m ? cand[q] : m;
    m = row16_max64(m);
#pragma unroll
    for (int q = 0; q < NE; ++q)
      if (cand[q] == m) cand[q] = 0ull;
    if (s == j) my_id = (int)~(uint32_t)m;
  }
  const float my_z = sel_value(z[my_id]);
  const float zmax = __shfl(my_z, lane & 48, 64);  // the group's first selection
  float denom = 1.f;
  if (a.gate == 0 || a.gate == 1) {  // softmax over the k selected / all E logits
    float acc = 0.f;
    if (a.gate == 0) {
      if (s < a.k) acc = expf(my_z - zmax);
    } else {
#pragma unroll
      for (int q = 0; q < NE; ++q) {
        const int e = q * 16 + s;
        if (e < a.E) acc += expf(sel_value(z[e]) - zmax);
      }
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) acc += __shfl_xor(acc, o, 64);
    denom = acc;
  }
  if (s < a.k && t < a.T) {
    const float wj = (a.gate == 2) ? sigmoid_f(my_z) : expf(my_z - zmax) / denom;
    const size_t o = (size_t)t * a.k + s;
    a.idx[o] = my_id;
    a.tw[o] = wj;
    a.local[o] = lmap[my_id];
  }
}

// Which logits path a block takes: STAGED4 / STAGED8 bf16, up to 64 experts
// and d <= 64 * 4 / 64 * 8 * RT_WAVES; DIRECT bf16, up to 64 experts, longer d;
// RING bf16 beyond 64 experts; F32 fp32 with 16-byte aligned rows, F32_DWORD
// fp32 otherwise.
enum RoutePath { STAGED4, STAGED8, DIRECT, RING, F32, F32_DWORD };

template <int NEB, int PATH>
__global__ __launch_bounds__(RT_THREADS) void route_fwd_kernel(RouteFwdArgs a) {
  constexpr int LDZ = NEB * 32 + 1;
  constexpr int NQ = (NEB * 32 + 63) / 64;  // logits (and selections) per lane
  __shared__ float zl[RT_TOK * LDZ];
  __shared__ int lmap[256];
  const int t0 = blockIdx.x * RT_TOK;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  if (wave == 0) build_local_map(a.resident, a.E, lmap);
  // every path ends with a barrier
  if constexpr (PATH == STAGED4) logits_mfma_staged<NEB, 4>(a, t0, zl, LDZ);
  else if constexpr (PATH == STAGED8) logits_mfma_staged<NEB, 8>(a, t0, zl, LDZ);
  else if constexpr (PATH == DIRECT) logits_mfma<NEB>(a, t0, zl, LDZ);
  else if constexpr (PATH == RING) logits_ring<NEB>(a, t0, zl, LDZ);
  else logits_f32<NEB * 32, PATH == F32>(a, t0, zl, LDZ);

  if (a.k <= RT_KSEL) {
    static_assert(RT_TOK == 4 * RT_WAVES, "16 lanes per token in every wave");
    select_groups<LDZ, 2 * NEB>(a, zl, t0, lmap);
    return;
  }
  for (int i = wave; i < RT_TOK; i += RT_WAVES) {
    const int t = t0 + i;
    if (t >= a.T) break;
    float v[NQ];
    bool taken[NQ];
    int my_e[NQ];
    float my_z[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = q * 64 + lane;
      taken[q] = !(e < a.E);
      v[q] = (e < a.E) ? zl[i * LDZ + e] : 0.f;
      if (v[q] != v[q]) v[q] = -INFINITY;  // NaN ranks last; some expert is always picked
      my_e[q] = 0;
      my_z[q] = 0.f;
    }
    float zmax = 0.f;
    for (int j = 0; j < a.k; ++j) {
      float bv = -INFINITY;
      int be = 0x7fffffff;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int e = q * 64 + lane;
        if (!taken[q] && (v[q] > bv || (v[q] == bv && e < be))) { bv = v[q]; be = e; }
      }
      wave_argmax(bv, be);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (q * 64 + lane == be) taken[q] = true;
        if (q * 64 + lane == j) { my_e[q] = be; my_z[q] = bv; }
      }
      if (j == 0) zmax = bv;
    }
    // gate weights of the selected experts (selection j lives in lane j % 64)
    float denom = 1.f;
    if (a.gate == 0) {  // softmax over the k selected logits
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (q * 64 + lane < a.k) s += expf(my_z[q] - zmax);
      denom = wave_sum(s);
    } else if (a.gate == 1) {  // softmax over all E logits
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (q * 64 + lane < a.E) s += expf(v[q] - zmax);
      denom = wave_sum(s);
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int j = q * 64 + lane;
      if (j < a.k) {
        float wj;
        if (a.gate == 2) wj = sigmoid_f(my_z[q]);
        else wj = expf(my_z[q] - zmax) / denom;
        const size_t o = (size_t)t * a.k + j;
        a.idx[o] = my_e[q];
        a.tw[o] = wj;
        a.local[o] = lmap[my_e[q]];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Backward.  dz per token (wave per token, lane per expert), then
// dW_r = inv_tau * dz^T x as per-chunk partial sums reduced in a fixed order,
// and dx (+)= inv_tau * dz W_r.

struct RouteBwdArgs {
  const void* x;
  const void* w;
  const int32_t* idx;
  const float* tw;
  const float* logits;
  const float* dtw;
  float* dz;
  float* dw;
  float* db;
  void* dx;
  float* part_w;  // [n_chunks][E][d]
  float* part_b;  // [n_chunks][n_bparts][E], or NULL (no d_bias wanted)
  int T, d, E, k, gate, accumulate_dx, n_chunks;
  int n_bparts;   // d_bias partial sums per chunk
  float inv_tau;
  float part_scale;  // factor of the partial sums: 1, or inv_tau when the only
                     // chunk's are the results (part_w = dw, part_b = db)
};

constexpr int RB_CHUNK = 256;  // tokens per partial sum of dW_r

__global__ __launch_bounds__(256) void route_dz_kernel(RouteBwdArgs a) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= a.T) return;
  const size_t o = (size_t)t * a.k;
  // s = <w, dw> over the k routes (lane-parallel, fixed tree order)
  float s = 0.f;
  for (int j = lane; j < a.k; j += 64) s += a.tw[o + j] * a.dtw[o + j];
  s = wave_sum(s);
  // softmax over all E (at most 256): the row's logits are read once
  float z[4], zmax = 0.f, denom = 1.f;
  if (a.gate == 1) {
    float m = -INFINITY;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = q * 64 + lane;
      z[q] = e < a.E ? a.logits[(size_t)t * a.E + e] : -INFINITY;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q * 64 + lane < a.E) m = fmaxf(m, z[q]);
    zmax = wave_max(m);
    float acc = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q * 64 + lane < a.E) acc += z[q] = expf(z[q] - zmax);
    denom = wave_sum(acc);
  }
  // lane j holds route j's expert and the route's own share of the gradient
  // (k <= 64; with more, the lane of the expert looks its route up)
  const bool held = a.k <= 64;
  auto share = [&](int j) {
    const float wv = a.tw[o + j], dv = a.dtw[o + j];
    return a.gate == 0 ? wv * (dv - s) : a.gate == 2 ? dv * wv * (1.f - wv) : dv;
  };
  const int my_e = held && lane < a.k ? a.idx[o + lane] : -1;
  const float my_g = held && lane < a.k ? share(lane) : 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 64 + lane;
    if (q * 64 >= a.E) break;
    float g = 0.f;
    if (held) {
      for (int j = a.k - 1; j >= 0; --j) {
        const int ej = __builtin_amdgcn_readlane(my_e, j);
        const float gj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_g), j));
        if (ej == e) g = gj;
      }
    } else {
      for (int j = a.k - 1; j >= 0; --j)
        if (a.idx[o + j] == e) g = share(j);
    }
    if (e < a.E) {
      if (a.gate == 1) g = z[q] / denom * (g - s);
      a.dz[(size_t)t * a.E + e] = g;
    }
  }
}

// V = 4: 16 bytes per load and store (E d % 4 == 0, 16-byte aligned dw).
template <int V>
__global__ __launch_bounds__(256) void route_dw_reduce_kernel(RouteBwdArgs a) {
  // dW_r[i] = inv_tau * (((p_0[i] + p_1[i]) + p_2[i]) + ...); the chunk
  // loads of a thread are issued 8 at a time
  typedef __attribute__((__vector_size__(V * 4))) float vec;
  const size_t n = (size_t)a.E * a.d / V;
  const vec* part = reinterpret_cast<const vec*>(a.part_w);
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    vec s = {};
    int c = 0;
    for (; c + 8 <= a.n_chunks; c += 8) {
      vec v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(c + u) * n + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; c < a.n_chunks; ++c) s += part[(size_t)c * n + i];
    reinterpret_cast<vec*>(a.dw)[i] = s * a.inv_tau;
  }
  if (a.db && blockIdx.x == 0) {
    // d_bias[e] = inv_tau * sum of the (chunk, part) partials: four
    // consecutive ranges summed by four threads, then added in range order
    __shared__ float q4[4][64];
    const int np = a.n_chunks * a.n_bparts;
    for (int e0 = 0; e0 < a.E; e0 += 64) {
      const int e = e0 + (threadIdx.x & 63), q = threadIdx.x >> 6;
      const int pb = (int)((long)np * q / 4), pe = (int)((long)np * (q + 1) / 4);
      float s = 0.f;
      if (e < a.E) {
        int c = pb;
        for (; c + 8 <= pe; c += 8) {
          float v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = a.part_b[(size_t)(c + u) * a.E + e];
#pragma unroll
          for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; c < pe; ++c) s += a.part_b[(size_t)c * a.E + e];
      }
      q4[q][threadIdx.x & 63] = s;
      __syncthreads();
      if (q == 0 && e < a.E)
        a.db[e] = (((q4[0][threadIdx.x] + q4[1][threadIdx.x]) + q4[2][threadIdx.x]) +
                   q4[3][threadIdx.x]) * a.inv_tau;
      __syncthreads();
    }
  }
}

// bf16 router backward on MFMA (E <= 64): one block = 128 columns (the last
// ones may lie past d) x RB_CHUNK tokens, in sub-chunks of 64 tokens.  Per sub-chunk the
// block stages x[tokens, cols] and dz[tokens, 0..63] in LDS, the fp32 dz split
// into NP bf16 parts, and computes
//   dW partial[e, c] += sum_t (parts)[t, e] x[t, c]            (k = tokens)
//   dx[t, c] (+)= inv_tau * sum_e (parts)[t, e] W_r[e, c]       (k = experts)
// with v_mfma_f32_32x32x16_bf16; wave w owns columns 32w..32w+31 of both.
// The next sub-chunk's x and dz are loaded into registers while the current
// one is computed; the dx result is staged through LDS so that the update of
// dx reads and writes whole row segments.  The per-chunk dW partials, and
// one d_bias partial per block (its column block's share of the chunk's
// tokens, so that no block carries the whole chunk's bias sum: that made the
// blocks of column 0 the critical path, 15 us of about 50), are summed in a
// fixed order by route_dw_reduce_kernel.
constexpr int RBM_COLS = 128;
constexpr int RBM_SUB = 64;                   // tokens per sub-chunk
constexpr int RBM_XS = RBM_COLS * 2 + 64;     // x row stride (bytes): the 4 rows of
                                              // a transposed read on distinct banks
constexpr int RBM_ZS = 64 * 2 + 16;           // dz row stride: 16 rows of a 16-byte
                                              // read on distinct banks
constexpr int RBM_WS = RBM_COLS * 2 + 64;     // W_r row stride
constexpr int RBM_STG = RBM_COLS + 4;  // fp32 row stride of the staged dx update
static_assert(RBM_SUB * RBM_STG * 4 <= RBM_SUB * RBM_XS + 2 * RBM_SUB * RBM_ZS,
              "the staged dx update must fit over the x and dz tiles");
constexpr int RBM_XV = RBM_SUB * RBM_COLS / 8 / 256;  // 16-byte x vectors per thread
constexpr int RBM_ZV = RBM_SUB * 64 / 8 / 256;        // 8-expert dz groups per thread
static_assert(RBM_XV * 256 * 8 == RBM_SUB * RBM_COLS && RBM_ZV * 256 * 8 == RBM_SUB * 64,
              "staging split");

// v as a sum of NP bf16 values: |v - sum| <= 2^-17 |v| for 2, nothing left for 3
// (of |v| between 2^-109 and bf16's largest value; see overflowed).
template <int NP>
DEVI void split_bf16(float v, bf16_t* out) {
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    out[p] = (bf16_t)v;
    v -= (float)out[p];
  }
}

// The same over 8 values, to LDS: part p at dst + p stride.
template <int NP>
DEVI void store_split8(const float* v, char* dst, int stride) {
  bf16x8_t o[NP];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    bf16_t q[NP];
    split_bf16<NP>(v[u], q);
#pragma unroll
    for (int p = 0; p < NP; ++p) o[p][u] = q[p];
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) *reinterpret_cast<bf16x8_t*>(dst + p * stride) = o[p];
}

// Sums over dz in 3 bf16 parts are those of the fp32 dz while every operand is
// finite.  The parts of an infinite dz, or of one past bf16's range, cancel to NaN,
// and so does an infinite x or W_r against parts of either sign or zero.  Such sums
// are no finite numbers, so a wave that finds one among its own takes them again
// from the fp32 dz, on fp32 MFMAs (exact_dw, exact_dx).  5003 tokens, d = 1536,
// 256 experts 47.9 -> 48.7 us by the check; 3001 tokens, d = 776, 32 experts 18.6 -> 19.0.

// Whether any of the n values is infinite or NaN, in any lane.
template <int N, class V>
DEVI bool overflowed(const V* v, int n) {
  float s = 0.f;
  for (int i = 0; i < n; ++i)
#pragma unroll
    for (int r = 0; r < N; ++r) s += v[i][r];
  return __ballot(!(fabsf(s) <= 3.4028234e38f)) != 0;
}
DEVI f32x4_t exact_mfma(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
DEVI f32x16_t exact_mfma(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
// x[t, c], W_r[e, c] and dz[t, e]; 0 outside
DEVI float bf16_at(const bf16_t* p, int r, int rows, int c, int d) {
  return r < rows && c < d ? (float)p[(size_t)r * d + c] : 0.f;
}
DEVI float dz_at(const RouteBwdArgs& a, int t, int e) {
  return t < a.T && e < a.E ? a.dz[(size_t)t * a.E + e] : 0.f;
}
// dW[e, c] of the chunk's tokens into acc[i][j]: experts e0 + S i, columns c0 + S j,
// S = 16 or 32 of each.
template <int S, int NI, int NJ, class V>
DEVI void exact_dw(const RouteBwdArgs& a, int chunk, int e0, int c0, V (*acc)[NJ]) {
  const int l = threadIdx.x & (S - 1), g = (threadIdx.x & 63) / S;
  const bf16_t* x = static_cast<const bf16_t*>(a.x);
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = V{};
#pragma unroll 1
  for (int t = chunk * RB_CHUNK + g; t < (chunk + 1) * RB_CHUNK; t += 64 / S)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const float xv = bf16_at(x, t, a.T, c0 + S * j + l, a.d);
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i][j] = exact_mfma(xv, dz_at(a, t, e0 + S * i + l), acc[i][j]);
    }
}
// sum_e dz[t, e] W_r[e, c] into acc[i][j]: tokens t0 + S i, columns c0 + S j.
template <int S, int NI, int NJ, class V>
DEVI void exact_dx(const RouteBwdArgs& a, int t0, int c0, V (*acc)[NJ]) {
  const int l = threadIdx.x & (S - 1), g = (threadIdx.x & 63) / S;
  const bf16_t* w = static_cast<const bf16_t*>(a.w);
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = V{};
#pragma unroll 1
  for (int e = g; e < (a.E + 3) / 4 * 4; e += 64 / S)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const float wv = bf16_at(w, e, a.E, c0 + S * j + l, a.d);
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i][j] = exact_mfma(wv, dz_at(a, t0 + S * i + l, e), acc[i][j]);
    }
}

// NP = 2 where d % 128 == 0; ragged d takes 3 parts (nothing of dz is lost).
template <int NP>
__global__ __launch_bounds__(256, 2) void route_bwd_mfma_kernel(RouteBwdArgs a) {
  constexpr int ZB = RBM_SUB * RBM_ZS;  // bytes of one part of dz
  __shared__ __attribute__((aligned(16))) char lds[RBM_SUB * RBM_XS + NP * ZB + 64 * RBM_WS];
  char* xs = lds;
  char* zs = xs + RBM_SUB * RBM_XS;
  char* wl = zs + NP * ZB;
  const bf16_t* x = static_cast<const bf16_t*>(a.x);
  const bf16_t* w = static_cast<const bf16_t*>(a.w);
  bf16_t* dx = static_cast<bf16_t*>(a.dx);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int c0 = blockIdx.x * RBM_COLS;
  const int chunk = blockIdx.y;
  const int n_sub = min(RB_CHUNK, a.T - chunk * RB_CHUNK + RBM_SUB - 1) / RBM_SUB;
  const bool vec_dz = (a.E & 3) == 0 && ((uintptr_t)a.dz & 15) == 0;
  const u32x4_t zero4 = {0u, 0u, 0u, 0u};

  // W_r[0..63, c0..c0+127] (rows >= E are zero)
  for (int p = tid; p < 64 * (RBM_COLS / 8); p += 256) {
    const int e = p / (RBM_COLS / 8), c = (p % (RBM_COLS / 8)) * 8;
    *reinterpret_cast<u32x4_t*>(wl + e * RBM_WS + c * 2) =
        e < a.E && c0 + c < a.d ? *reinterpret_cast<const u32x4_t*>(w + (size_t)e * a.d + c0 + c) : zero4;
  }

  // register staging of one sub-chunk: thread owns x vectors p = tid + 256 v
  // (row p / 16, columns 8 (p % 16)..) and dz groups p = tid + 256 v (row p / 8,
  // experts 8 (p % 8)..)
  u32x4_t xr[RBM_XV];
  float zr[RBM_ZV][8];
  const bool col_ok = c0 + (tid & 15) * 8 < a.d;  // this thread's 8 columns
  auto load_sub = [&](int t0) {
#pragma unroll
    for (int v = 0; v < RBM_XV; ++v) {
      const int p = tid + 256 * v;
      const int t = t0 + (p >> 4);
      xr[v] = t < a.T && col_ok ? *reinterpret_cast<const u32x4_t*>(x + (size_t)t * a.d + c0 + (p & 15) * 8)
                      : zero4;
    }
#pragma unroll
    for (int v = 0; v < RBM_ZV; ++v) {
      const int p = tid + 256 * v;
      const int t = t0 + (p >> 3), e0 = (p & 7) * 8;
      const float* src = a.dz + (size_t)t * a.E + e0;
      if (t < a.T && vec_dz && e0 + 8 <= a.E) {
        const f32x4_t u0 = *reinterpret_cast<const f32x4_t*>(src);
        const f32x4_t u1 = *reinterpret_cast<const f32x4_t*>(src + 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) { zr[v][u] = u0[u]; zr[v][4 + u] = u1[u]; }
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) zr[v][u] = (t < a.T && e0 + u < a.E) ? src[u] : 0.f;
      }
    }
  };
  auto store_sub = [&]() {
#pragma unroll
    for (int v = 0; v < RBM_XV; ++v) {
      const int p = tid + 256 * v;
      *reinterpret_cast<u32x4_t*>(xs + (p >> 4) * RBM_XS + (p & 15) * 16) = xr[v];
    }
#pragma unroll
    for (int v = 0; v < RBM_ZV; ++v) {
      const int p = tid + 256 * v;
      store_split8<NP>(zr[v], zs + (p >> 3) * RBM_ZS + (p & 7) * 16, ZB);
    }
  };

  f32x16_t accw[2] = {f32x16_t{}, f32x16_t{}};
  if (n_sub > 0) load_sub(chunk * RB_CHUNK);
  // d_bias partial: column block b < n_bparts sums the exact fp32 dz of the
  // sub-chunks s with s % n_bparts == b, from the registers that stage them:
  // per thread its two rows, then across the 8 lanes of an expert group
  // (xor shuffles), then (at the end) across the 4 waves in wave order
  const bool do_bias = a.part_b && (int)blockIdx.x < a.n_bparts;
  float bacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int sc = 0; sc < n_sub; ++sc) {
    const int t0 = chunk * RB_CHUNK + sc * RBM_SUB;
    __syncthreads();  // previous sub-chunk's LDS reads are done
    store_sub();
    if (do_bias && sc % a.n_bparts == (int)blockIdx.x) {
      static_assert(RBM_ZV == 2, "two dz rows per thread");
      float b8[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) b8[u] = zr[0][u] + zr[1][u];
#pragma unroll
      for (int m = 8; m < 64; m <<= 1)
#pragma unroll
        for (int u = 0; u < 8; ++u) b8[u] += __shfl_xor(b8[u], m, 64);
#pragma unroll
      for (int u = 0; u < 8; ++u) bacc[u] += b8[u];
    }
    __syncthreads();
    if (sc + 1 < n_sub) load_sub(t0 + RBM_SUB);
    // old dx of this thread's 16-byte chunks of the sub-chunk (requested
    // before the MFMAs; used by the coalesced update below)
    u32x4_t old[RBM_XV];
    if (a.accumulate_dx && col_ok) {
#pragma unroll
      for (int v = 0; v < RBM_XV; ++v) {
        const int p = tid + 256 * v;
        const int t = min(t0 + (p >> 4), a.T - 1);
        old[v] = *reinterpret_cast<const u32x4_t*>(dx + (size_t)t * a.d + c0 + (p & 15) * 8);
      }
    }

    // dW partial: k = tokens, m = experts (2 blocks), n = columns
#pragma unroll
    for (int ks = 0; ks < RBM_SUB / 16; ++ks) {
      const bf16x8_t bx = frag_tr(xs, RBM_XS, ks * 16, wave * 32);
#pragma unroll
      for (int eb = 0; eb < 2; ++eb) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
          accw[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              bx, frag_tr(zs + p * ZB, RBM_ZS, ks * 16, eb * 32), accw[eb], 0, 0, 0);
      }
    }

    // dx: k = experts (4 k16-steps), m = tokens (2 blocks), n = columns
    f32x16_t accx[2] = {f32x16_t{}, f32x16_t{}};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const bf16x8_t bw = frag_tr(wl, RBM_WS, ks * 16, wave * 32);
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const int r = tb * 32 + (lane & 31);
        const int e = ks * 16 + 8 * (lane >> 5);
#pragma unroll
        for (int p = 0; p < NP; ++p)
          accx[tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              bw, *reinterpret_cast<const bf16x8_t*>(zs + p * ZB + r * RBM_ZS + e * 2), accx[tb], 0, 0, 0);
      }
    }
    if constexpr (NP == 3) {
      if (overflowed<16>(accx, 2))
        exact_dx<32, 2, 1>(a, t0, c0 + wave * 32, reinterpret_cast<f32x16_t(*)[1]>(accx));
    }
    // lane holds dx[t0 + 32 tb + lane%32][c0 + 32 wave + 8q + 4(lane/32) + 0..3];
    // staged as fp32 through LDS (over the x and dz tiles, now consumed) so
    // that the update of dx reads and writes whole 256-byte row segments
    __syncthreads();
    float* stg = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4_t v = {accx[tb][4 * q], accx[tb][4 * q + 1], accx[tb][4 * q + 2],
                           accx[tb][4 * q + 3]};
        *reinterpret_cast<f32x4_t*>(stg + (tb * 32 + (lane & 31)) * RBM_STG +
                                    wave * 32 + 8 * q + 4 * (lane >> 5)) = v;
      }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < RBM_XV; ++v) {
      const int p = tid + 256 * v;
      const int r = p >> 4, c = (p & 15) * 8;
      const int t = t0 + r;
      if (t >= a.T || !col_ok) continue;
      const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(stg + r * RBM_STG + c);
      const f32x4_t hi = *reinterpret_cast<const f32x4_t*>(stg + r * RBM_STG + c + 4);
      const bf16x8_t ob = __builtin_bit_cast(bf16x8_t, old[v]);
      bf16x8_t o;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float add = a.inv_tau * (u < 4 ? lo[u] : hi[u - 4]);
        o[u] = (bf16_t)(a.accumulate_dx ? (float)ob[u] + add : add);
      }
      *reinterpret_cast<bf16x8_t*>(dx + (size_t)t * a.d + c0 + c) = o;
    }
  }

  if constexpr (NP == 3) {
    if (overflowed<16>(accw, 2))
      exact_dw<32, 2, 1>(a, chunk, 0, c0 + wave * 32, reinterpret_cast<f32x16_t(*)[1]>(accw));
  }
  // lane holds partial[e = 32 eb + lane%32][c0 + 32 wave + 8q + 4(lane/32) + 0..3]
#pragma unroll
  for (int eb = 0; eb < 2; ++eb) {
    const int e = eb * 32 + (lane & 31);
    if (e >= a.E) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (c0 + wave * 32 + 8 * q + 4 * (lane >> 5) >= a.d) continue;
      float* p = a.part_w + ((size_t)chunk * a.E + e) * a.d + c0 + wave * 32 + 8 * q +
                 4 * (lane >> 5);
      const f32x4_t o = {accw[eb][4 * q], accw[eb][4 * q + 1], accw[eb][4 * q + 2],
                         accw[eb][4 * q + 3]};
      *reinterpret_cast<f32x4_t*>(p) = o * a.part_scale;
    }
  }
  if (do_bias) {
    // lanes 0..7 hold experts 8 lane .. 8 lane + 7 of this wave's rows
    __shared__ float bpart[4][64];
    if (lane < 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) bpart[wave][lane * 8 + u] = bacc[u];
    __syncthreads();
    if (tid < a.E)
      a.part_b[((size_t)chunk * a.n_bparts + blockIdx.x) * a.E + tid] =
          (((bpart[0][tid] + bpart[1][tid]) + bpart[2][tid]) + bpart[3][tid]) * a.part_scale;
  }
}

// d_bias partial of this block: rows[r][e], r < R (EP experts each, in LDS), are
// its threads' shares; added in row order.
template <int EP, int R>
DEVI void store_bias(const RouteBwdArgs& a, int chunk, const float* rows) {
  if ((int)threadIdx.x >= a.E) return;
  float s = 0.f;
#pragma unroll 8
  for (int r = 0; r < R; ++r) s += rows[r * EP + threadIdx.x];
  a.part_b[((size_t)chunk * a.n_bparts + blockIdx.x) * a.E + threadIdx.x] = s * a.part_scale;
}

// 8 (or 4) experts e0.. of dz row t into v; zeros past E and T.
template <int N>
DEVI void load_dz(const RouteBwdArgs& a, int t, int e0, bool vec, float* v) {
  const float* src = a.dz + (size_t)t * a.E + e0;
  if (t < a.T && vec && e0 + N <= a.E) {
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {
      const f32x4_t u = *reinterpret_cast<const f32x4_t*>(src + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * q + e] = u[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = t < a.T && e0 + e < a.E ? src[e] : 0.f;
  }
}

// v_mfma_f32_16x16x32 operand fragment (lane l: index i0 + l % 16, k = k0 +
// 8 (l / 16) + 0..7) of an LDS array whose rows are k (see frag_tr).
DEVI bf16x8_t frag_tr16(const char* base, int stride, int k0, int i0) {
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, i = lane & 15;
  s16x4_t v[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(
        base + (size_t)(k0 + 8 * g + 4 * h + (i >> 2)) * stride + (i0 + 4 * (i & 3)) * 2));
  const s16x8_t both = __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, both);
}

constexpr int RBW_COLS = 64;  // columns per block of the two kernels below

// The same for 65 to 256 experts (EP = 128 or 256): 8 waves, 64 columns x
// RB_CHUNK tokens, all EP experts of W_r's columns and of 64 tokens' dz in LDS.
// Wave (quarter, half) computes dW of a quarter of the experts and dx of a
// quarter of the tokens, for half of the columns, on 16 x 16 x 32 MFMAs with dz
// in 3 bf16 parts (its whole fp32 value).  5003 tokens, d = 1536, 256 experts:
// 49 us; the VALU kernels this replaces took 364 (dW partials) + 108 us (dx),
// bound by their LDS and L2 operand reads.
template <int EP>
__global__ __launch_bounds__(512) void route_bwd_wide_kernel(RouteBwdArgs a) {
  constexpr int SUB = RBM_SUB, XS = RBW_COLS * 2 + 32, ZS = EP * 2 + 16;
  constexpr int G = EP / 8, ZR = 512 / G, ZV = SUB / ZR;  // dz: 8-expert groups, rows per pass, passes
  constexpr int EQ = EP / 4, ET = EQ / 16;
  constexpr int NP = 3, ZB = SUB * ZS;  // parts of dz, bytes of one
  __shared__ __attribute__((aligned(16))) char lds[SUB * XS + NP * ZB + EP * XS];
  char* xs = lds;
  char* zs = xs + SUB * XS;
  char* wl = zs + NP * ZB;
  static_assert(ZR * EP * 4 <= NP * ZB, "the bias shares fit over dz");
  const bf16_t* x = static_cast<const bf16_t*>(a.x);
  const bf16_t* w = static_cast<const bf16_t*>(a.w);
  bf16_t* dx = static_cast<bf16_t*>(a.dx);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int quarter = wave >> 1, col0 = (wave & 1) * 32;
  const int c0 = blockIdx.x * RBW_COLS, chunk = blockIdx.y;
  const int n_sub = (min(RB_CHUNK, a.T - chunk * RB_CHUNK) + SUB - 1) / SUB;
  const bool vec_dz = (a.E & 3) == 0 && ((uintptr_t)a.dz & 15) == 0;
  const u32x4_t zero4 = {0u, 0u, 0u, 0u};
  for (int p = tid; p < EP * 8; p += 512) {
    const int e = p >> 3, c = (p & 7) * 8;
    *reinterpret_cast<u32x4_t*>(wl + e * XS + c * 2) =
        e < a.E && c0 + c < a.d ? *reinterpret_cast<const u32x4_t*>(w + (size_t)e * a.d + c0 + c) : zero4;
  }
  u32x4_t xr;
  float zr[ZV][8];
  auto load_sub = [&](int t0) {
    const int t = t0 + (tid >> 3), c = c0 + (tid & 7) * 8;
    xr = t < a.T && c < a.d ? *reinterpret_cast<const u32x4_t*>(x + (size_t)t * a.d + c) : zero4;
#pragma unroll
    for (int v = 0; v < ZV; ++v) load_dz<8>(a, t0 + tid / G + v * ZR, tid % G * 8, vec_dz, zr[v]);
  };
  auto store_sub = [&]() {
    *reinterpret_cast<u32x4_t*>(xs + (tid >> 3) * XS + (tid & 7) * 16) = xr;
#pragma unroll
    for (int v = 0; v < ZV; ++v)
      store_split8<NP>(zr[v], zs + (tid / G + v * ZR) * ZS + tid % G * 16, ZB);
  };
  f32x4_t accw[ET][2];
#pragma unroll
  for (int i = 0; i < ET; ++i) accw[i][0] = accw[i][1] = f32x4_t{};
  const bool do_bias = a.part_b && (int)blockIdx.x < a.n_bparts;
  float bacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  load_sub(chunk * RB_CHUNK);
  for (int sc = 0; sc < n_sub; ++sc) {
    const int t0 = chunk * RB_CHUNK + sc * SUB;
    __syncthreads();  // the previous sub-chunk's LDS reads are done
    store_sub();
    if (do_bias && sc % a.n_bparts == (int)blockIdx.x)
#pragma unroll
      for (int v = 0; v < ZV; ++v)
#pragma unroll
        for (int u = 0; u < 8; ++u) bacc[u] += zr[v][u];
    __syncthreads();
    if (sc + 1 < n_sub) load_sub(t0 + SUB);
    const int t = t0 + quarter * 16 + l16;
    bf16x4_t old[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = c0 + col0 + 16 * j + 4 * g4;
      if (a.accumulate_dx && t < a.T && c < a.d)
        old[j] = *reinterpret_cast<const bf16x4_t*>(dx + (size_t)t * a.d + c);
    }
#pragma unroll
    for (int ks = 0; ks < SUB / 32; ++ks) {  // dW: k = tokens
      bf16x8_t xf[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) xf[j] = frag_tr16(xs, XS, ks * 32, col0 + 16 * j);
#pragma unroll
      for (int i = 0; i < ET; ++i) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const bf16x8_t zf = frag_tr16(zs + p * ZB, ZS, ks * 32, quarter * EQ + 16 * i);
#pragma unroll
          for (int j = 0; j < 2; ++j)
            accw[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[j], zf, accw[i][j], 0, 0, 0);
        }
      }
    }
    f32x4_t accx[2] = {f32x4_t{}, f32x4_t{}};
#pragma unroll
    for (int ks = 0; ks < EP / 32; ++ks) {  // dx: k = experts
      const char* zrow = zs + (quarter * 16 + l16) * ZS + (ks * 32 + 8 * g4) * 2;
      bf16x8_t wf[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) wf[j] = frag_tr16(wl, XS, ks * 32, col0 + 16 * j);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const bf16x8_t zf = *reinterpret_cast<const bf16x8_t*>(zrow + p * ZB);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          accx[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], zf, accx[j], 0, 0, 0);
      }
    }
    if (overflowed<4>(accx, 2))
      exact_dx<16, 1, 2>(a, t0 + quarter * 16, c0 + col0, &accx);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = c0 + col0 + 16 * j + 4 * g4;
      if (t >= a.T || c >= a.d) continue;
      bf16x4_t o;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float add = a.inv_tau * accx[j][u];
        o[u] = (bf16_t)(a.accumulate_dx ? (float)old[j][u] + add : add);
      }
      *reinterpret_cast<bf16x4_t*>(dx + (size_t)t * a.d + c) = o;
    }
  }
  if (overflowed<4>(&accw[0][0], 2 * ET)) exact_dw<16, ET, 2>(a, chunk, quarter * EQ, c0 + col0, accw);
#pragma unroll
  for (int i = 0; i < ET; ++i) {
    const int e = quarter * EQ + 16 * i + l16;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = c0 + col0 + 16 * j + 4 * g4;
      if (e < a.E && c < a.d)
        *reinterpret_cast<f32x4_t*>(a.part_w + ((size_t)chunk * a.E + e) * a.d + c) =
            accw[i][j] * a.part_scale;
    }
  }
  if (do_bias) {
    __syncthreads();
    float* rows = reinterpret_cast<float*>(zs);
#pragma unroll
    for (int u = 0; u < 8; ++u) rows[tid / G * EP + tid % G * 8 + u] = bacc[u];
    __syncthreads();
    store_bias<EP, ZR>(a, chunk, rows);
  }
}

// Router backward of fp32 layers on v_mfma_f32_16x16x4_f32: 4 waves, 64 columns
// x RB_CHUNK tokens in sub-chunks of 64, EP (16, 64, 128 or 256) experts in LDS.
// Wave w computes 16 columns of dW (MFMA tile i of expert block b: experts 64 b
// + MI (l % 16) + i, so a lane reads MI consecutive ones) and of dx.  The VALU
// kernels this replaces waited out a memory latency per 32 tokens: 256 tokens,
// d = 64, 8 experts took 49 (dW) + 5 us (dx), now 10.
template <int EP>
__global__ __launch_bounds__(256) void route_bwd_f32_kernel(RouteBwdArgs a) {
  constexpr int SUB = RBM_SUB, XS = RBW_COLS + 4, ZS = EP + 4;  // row strides (floats)
  constexpr int MI = EP >= 64 ? 4 : 1, EB = EP / (16 * MI);
  constexpr int G = EP / 4, ZR = 256 / G, ZV = SUB / ZR;  // dz: 4-expert groups, rows per pass, passes
  __shared__ __attribute__((aligned(16))) float lds[SUB * XS + SUB * ZS + EP * XS];
  float* xs = lds;
  float* zs = xs + SUB * XS;
  float* wl = zs + SUB * ZS;
  static_assert(ZR * EP <= SUB * XS, "the bias shares fit over x");
  const float* x = static_cast<const float*>(a.x);
  const float* w = static_cast<const float*>(a.w);
  float* dx = static_cast<float*>(a.dx);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int c0 = blockIdx.x * RBW_COLS, chunk = blockIdx.y;
  const int n_sub = (min(RB_CHUNK, a.T - chunk * RB_CHUNK) + SUB - 1) / SUB;
  const bool vec_dz = (a.E & 3) == 0 && ((uintptr_t)a.dz & 15) == 0;
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  const int col = c0 + (tid & 15) * 4;  // this thread's columns of x and W_r
  f32x4_t xr[4];
  float zr[ZV][4];
  auto load_sub = [&](int t0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int t = t0 + (tid >> 4) + 16 * v;
      xr[v] = t < a.T && col < a.d ? *reinterpret_cast<const f32x4_t*>(x + (size_t)t * a.d + col) : zero;
    }
#pragma unroll
    for (int v = 0; v < ZV; ++v) load_dz<4>(a, t0 + tid / G + v * ZR, tid % G * 4, vec_dz, zr[v]);
  };
  load_sub(chunk * RB_CHUNK);
#pragma unroll 4
  for (int e = tid >> 4; e < EP; e += 16)
    *reinterpret_cast<f32x4_t*>(wl + e * XS + (tid & 15) * 4) =
        e < a.E && col < a.d ? *reinterpret_cast<const f32x4_t*>(w + (size_t)e * a.d + col) : zero;
  f32x4_t accw[EB][MI];
#pragma unroll
  for (int b = 0; b < EB; ++b)
#pragma unroll
    for (int i = 0; i < MI; ++i) accw[b][i] = zero;
  const bool do_bias = a.part_b && (int)blockIdx.x < a.n_bparts;
  f32x4_t bacc = zero;
  const int oc = c0 + wave * 16 + 4 * g4;  // the lane's 4 output columns
  for (int sc = 0; sc < n_sub; ++sc) {
    const int t0 = chunk * RB_CHUNK + sc * SUB;
    __syncthreads();  // the previous sub-chunk's LDS reads are done
#pragma unroll
    for (int v = 0; v < 4; ++v)
      *reinterpret_cast<f32x4_t*>(xs + ((tid >> 4) + 16 * v) * XS + (tid & 15) * 4) = xr[v];
#pragma unroll
    for (int v = 0; v < ZV; ++v) {
      const f32x4_t z = {zr[v][0], zr[v][1], zr[v][2], zr[v][3]};
      *reinterpret_cast<f32x4_t*>(zs + (tid / G + v * ZR) * ZS + tid % G * 4) = z;
      if (do_bias && sc % a.n_bparts == (int)blockIdx.x) bacc += z;
    }
    __syncthreads();
    if (sc + 1 < n_sub) load_sub(t0 + SUB);
    f32x4_t old[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + 16 * i + l16;
      if (a.accumulate_dx && t < a.T && oc < a.d)
        old[i] = *reinterpret_cast<const f32x4_t*>(dx + (size_t)t * a.d + oc);
    }
#pragma unroll 4
    for (int s = 0; s < SUB / 4; ++s) {  // dW: k = tokens
      const int k = 4 * s + g4;
      const float xv = xs[k * XS + wave * 16 + l16];
#pragma unroll
      for (int b = 0; b < EB; ++b) {
        typedef __attribute__((__vector_size__(MI * 4))) float vM;
        const vM zv = *reinterpret_cast<const vM*>(zs + k * ZS + 64 * b + MI * l16);
#pragma unroll
        for (int i = 0; i < MI; ++i)
          accw[b][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv, zv[i], accw[b][i], 0, 0, 0);
      }
    }
    f32x4_t accx[4] = {zero, zero, zero, zero};
#pragma unroll 2
    for (int q = 0; q < EP / 16; ++q) {  // dx: k = experts
      f32x4_t zv[4];
      float wv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        zv[i] = *reinterpret_cast<const f32x4_t*>(zs + (16 * i + l16) * ZS + 16 * q + 4 * g4);
#pragma unroll
      for (int e = 0; e < 4; ++e) wv[e] = wl[(16 * q + 4 * g4 + e) * XS + wave * 16 + l16];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          accx[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[e], zv[i][e], accx[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + 16 * i + l16;
      if (t >= a.T || oc >= a.d) continue;
      f32x4_t v = accx[i] * a.inv_tau;
      if (a.accumulate_dx) v += old[i];
      *reinterpret_cast<f32x4_t*>(dx + (size_t)t * a.d + oc) = v;
    }
  }
#pragma unroll
  for (int b = 0; b < EB; ++b)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int e = 64 * b + MI * l16 + i;
      if (e < a.E && oc < a.d)
        *reinterpret_cast<f32x4_t*>(a.part_w + ((size_t)chunk * a.E + e) * a.d + oc) =
            accw[b][i] * a.part_scale;
    }
  if (do_bias) {
    __syncthreads();
    *reinterpret_cast<f32x4_t*>(xs + tid / G * EP + tid % G * 4) = bacc;
    __syncthreads();
    store_bias<EP, ZR>(a, chunk, xs);
  }
}

}  // namespace

hipError_t launch_route_fwd(const void* x, const void* w, const float* bias, int bf16, int T,
                            int d, int E, int k, float inv_tau, int gate, const uint8_t* resident,
                            float* logits, int32_t* idx, float* tw, int32_t* local,
                            hipStream_t s) {
  RouteFwdArgs a{x, w, bias, resident, logits, idx, tw, local, T, d, E, k, gate, inv_tau};
  if (T == 0) return hipSuccess;
  const dim3 grid(ceil_div(T, RT_TOK));
  const int neb = E <= 32 ? 1 : E <= 64 ? 2 : E <= 128 ? 4 : 8;
  const bool vec = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w)) & 15) == 0;
#define ROUTE_LAUNCH(N, P) MOE_TIMED("route_fwd", s, route_fwd_kernel<N, P><<<grid, RT_THREADS, 0, s>>>(a))
#define ROUTE_F32(N)                       \
  do {                                     \
    if (vec) ROUTE_LAUNCH(N, F32);    \
    else ROUTE_LAUNCH(N, F32_DWORD);  \
  } while (0)
#define ROUTE_BF16(N)                                        \
  do {                                                       \
    if (d <= 64 * 4 * RT_WAVES) ROUTE_LAUNCH(N, STAGED4);    \
    else if (d <= 64 * 8 * RT_WAVES) ROUTE_LAUNCH(N, STAGED8); \
    else ROUTE_LAUNCH(N, DIRECT);                            \
  } while (0)
  switch (neb) {
    case 1:
      if (bf16) ROUTE_BF16(1);
      else ROUTE_F32(1);
      break;
    case 2:
      if (bf16) ROUTE_BF16(2);
      else ROUTE_F32(2);
      break;
    case 4:
      if (bf16) ROUTE_LAUNCH(4, RING);
      else ROUTE_F32(4);
      break;
    default:
      if (bf16) ROUTE_LAUNCH(8, RING);
      else ROUTE_F32(8);
      break;
  }
#undef ROUTE_LAUNCH
#undef ROUTE_F32
#undef ROUTE_BF16
  return hipGetLastError();
}

// d_bias partial sums per chunk: one per 64-token sub-chunk (at most one per 128
// columns)
int route_bwd_bparts(int d) { return std::max(1, std::min(d / RBM_COLS, RB_CHUNK / RBM_SUB)); }

size_t route_bwd_ws_bytes(int T, int d, int E) {
  const size_t chunks = (size_t)(T + RB_CHUNK - 1) / RB_CHUNK;
  return chunks * (size_t)E * ((size_t)d + route_bwd_bparts(d)) * sizeof(float) + 256;
}

hipError_t launch_route_bwd(const void* x, const void* w, int bf16, int T, int d, int E, int k,
                            float inv_tau, int gate, const int32_t* idx, const float* tw,
                            const float* logits, const float* dtw, float* dz, float* dw_router,
                            float* d_bias, void* dx, int accumulate_dx, void* ws,
                            hipStream_t s) {
  const int n_chunks = (T + RB_CHUNK - 1) / RB_CHUNK;
  const bool dw_vec = (reinterpret_cast<uintptr_t>(dw_router) & 15) == 0;
  // a single chunk's sums are the results: no partials, no reduction
  const bool direct = n_chunks == 1 && dw_vec;
  float* part_w = direct ? dw_router : static_cast<float*>(ws);
  float* part_b = !d_bias ? nullptr : direct ? d_bias : part_w + (size_t)n_chunks * E * d;
  RouteBwdArgs a{x, w, idx, tw, logits, dtw, dz, dw_router, d_bias, dx, part_w, part_b,
                 T, d, E, k, gate, accumulate_dx, n_chunks, direct ? 1 : route_bwd_bparts(d),
                 inv_tau, direct ? inv_tau : 1.f};
  if (T > 0) {
    MOE_TIMED("route_dz", s, route_dz_kernel<<<ceil_div(T, 4), 256, 0, s>>>(a));
    const dim3 g128(ceil_div(d, RBM_COLS), n_chunks), g64(ceil_div(d, RBW_COLS), n_chunks);
    if (bf16) {
      if (E <= 64 && d % RBM_COLS == 0)
        MOE_TIMED("route_bwd_mfma", s, route_bwd_mfma_kernel<2><<<g128, 256, 0, s>>>(a));
      else if (E <= 64) MOE_TIMED("route_bwd_mfma", s, route_bwd_mfma_kernel<3><<<g128, 256, 0, s>>>(a));
      else if (E <= 128) MOE_TIMED("route_bwd_wide", s, route_bwd_wide_kernel<128><<<g64, 512, 0, s>>>(a));
      else MOE_TIMED("route_bwd_wide", s, route_bwd_wide_kernel<256><<<g64, 512, 0, s>>>(a));
    } else {
      if (E <= 16) MOE_TIMED("route_bwd_f32", s, route_bwd_f32_kernel<16><<<g64, 256, 0, s>>>(a));
      else if (E <= 64) MOE_TIMED("route_bwd_f32", s, route_bwd_f32_kernel<64><<<g64, 256, 0, s>>>(a));
      else if (E <= 128) MOE_TIMED("route_bwd_f32", s, route_bwd_f32_kernel<128><<<g64, 256, 0, s>>>(a));
      else MOE_TIMED("route_bwd_f32", s, route_bwd_f32_kernel<256><<<g64, 256, 0, s>>>(a));
    }
  }
  if (!direct) {
    // n_chunks == 0 (T == 0) sums nothing and writes zeros.  16 bytes per
    // access once that still gives every CU a block (256 experts x 1536: 12.3
    // us with 4-byte accesses).
    const size_t n = (size_t)E * d;
    if (dw_vec && n >= (size_t)4 * 256 * 256) {
      const int blocks = (int)std::min<size_t>(4096, (n / 4 + 255) / 256);
      MOE_TIMED("route_dw_reduce", s, route_dw_reduce_kernel<4><<<blocks, 256, 0, s>>>(a));
    } else {
      const int blocks = (int)std::min<size_t>(4096, (n + 255) / 256);
      MOE_TIMED("route_dw_reduce", s, route_dw_reduce_kernel<1><<<blocks, 256, 0, s>>>(a));
    }
  }
  return hipGetLastError();
}

}  // namespace moe
