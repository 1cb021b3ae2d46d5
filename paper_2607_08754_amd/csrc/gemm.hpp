// GEMM core of the Polar Express step (device code, included by kernels.hip).
// One launch covers every matrix of the set: each block takes one output tile
// from the launch's tile list.
//
//   Gram    A  = X X^T                 NT: both operands are rows of X (k = Q)
//   Poly    B  = b A + c A A^T + a I   NT on the symmetric A (A A^T = A A); the
//                                      a X term of the step is folded into B
//   Update  X' = B X                   B symmetric (rows of B = columns of B);
//                                      X is read as [k][n].
//                                      Cubic steps (no Poly) use X' = a X + b A X
//                                      with the a X term in the epilogue.
//   Last    X_T = B X, stored like an update, with the per-tile partial
//           sums of X_0' * P over the canonical tile: P = X_T as stored
//           (rounded to the iterate type, the values the gradient kernel
//           reads) and X_0' = W / 2^e as stored, so that 2^e times the sum
//           is the trace sum(W * P) of Sec. 3
//
// The first step runs on X_0' = W / 2^e and applies kappa = 2^e / (f + eps)
// through its coefficients (per matrix: kappa a, kappa^3 b, kappa^5 c). Split sets
// with eps > 0 hold every iterate in a power of two of its own (step_scale).
//
// Gram and Poly outputs are symmetric: only tiles with tm <= tn are computed
// and off-diagonal tiles are also stored transposed (mirror).
//
// This file holds what the kernels share and k_gemm, the products on fp32
// MFMA: fp32 sets whose table the split form does not fit, and those whose
// gradients are bf16. gemm_pipe.hpp has the products on 16-bit operands.
//
// k_gemm's LDS layout: each operand row of a k-slab is 128 bytes (32 values
// of consecutive k) split into eight 16-byte chunks stored at chunk index
// c ^ key(row). A wave's 16-byte fragment reads touch 8 consecutive
// rows per 8-lane phase, which then land in 8 distinct bank groups; the
// stores of the transposing loader (16 lanes per row) are conflict-free too.
// Two LDS stages, one barrier per k-slab: the K-major operands go
// global -> LDS directly, the [k][n] operand is loaded into registers and
// stored transposed; the loads of slab k + 1 are in flight while the MFMAs of
// slab k run.
// Included inside namespace slorr, after the helpers of kernels.hip.
#pragma once

// fp32 MFMA. A lane feeds 16 bytes of one row of each operand (4 consecutive
// k); lanes 0-31 and 32-63 take the two halves of an 8 wide k step. Both
// operands use the same lane -> k map, so the instruction's internal k order
// does not matter for the sum.
struct Mfma {
  typedef float4v frag;
  static constexpr int V = 4;
  __device__ static __forceinline__ void mma(floatx16 &c, const frag &a, const frag &b) {
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1], b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[2], b[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[3], b[3], c, 0, 0, 0);
  }
};

enum GemmMode { kGram = 0, kPoly = 1, kUpdate = 2, kLast = 3 };

struct GemmArgs {
  const Tile *tiles;
  const MatDesc *mats;
  const DynDesc *dyn;
  char *ws;
  double *tpart;
  const Scalars *sc;
  int xin, xout;  // X buffers read / written (MatDesc::x index)
  int use_a;      // update operand is A (cubic step)
  int write_x;    // Last: store X_T (the gradient kernel reads it)
  int fold;       // Update / Last: a_t I is folded into the operand (no a X term)
  int kap;        // coefficients per matrix (step_scale): kKappa in the first step, kRescale
  int grow0, grow1;  // Launch::grow0, grow1
  float alpha, beta, gamma;
  float *gpart;   // Gram parts (split K): fp32 partial tiles, BM x BN each, at tile.slot
  int quads;      // k_upd256 over a list of 128-tiles: a trace slot per 128 x 128 quadrant
                  // (slot of the first, Pp / 128 slots from one column of quadrants to the next)
  int ntiles;     // entries of the tile list (a persistent kernel's grid can be smaller)
};

// The step's coefficients for the iterate as it is held: X_t = k X^_t, so that
// X^' = m (a + b k^2 A^ + c k^4 A^^2) X^ with m = k over the next iterate's k.
// First step: k = kappa 2^-h, all others 2^-h_t (see Scalars).
enum KapBits { kKappa = 1, kRescale = 2 };
struct StepScale {
  double k2, m;
};
__device__ __forceinline__ StepScale step_scale(const GemmArgs &a, int mat) {
  const Scalars &s = a.sc[mat];
  double k = a.kap & kKappa ? s.kappa : 1.0, m = k;
  if (a.kap & kRescale) {
    const int h0 = max(0, s.shift - a.grow0), h1 = max(0, s.shift - a.grow1);
    k = ldexp(k, -h0);
    m = ldexp(m, h1 - h0);
  }
  return {k * k, m};
}

template <int BM, int BN, int WGM, int WGN>
struct GemmShape {
  static constexpr int kWaves = WGM * WGN;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int WTM = BM / WGM, WTN = BN / WGN;   // wave tile
  static constexpr int FM = WTM / 32, FN = WTN / 32;     // 32x32 MFMA tiles per wave
  static constexpr int kStage = (BM + BN) * 128;         // bytes per LDS stage
  static constexpr int kEpiPitch = WTN + 4;              // floats per staged row
  static constexpr int kEpiWave = 32 * kEpiPitch * 4;    // staged bytes per wave
  static constexpr int kEpiAll = kWaves * kEpiWave;
  static constexpr int kSmem = (2 * kStage > kEpiAll) ? 2 * kStage : kEpiAll;
};

// Byte offset of 16-byte chunk `chunk` of LDS row `row`. The XOR key
// (row & 7) ^ ((row >> 3) & 1) permutes the chunks so that (a) any 8
// consecutive rows (one 8-lane phase of a 16-byte read with 32 banks) use 8
// distinct chunk positions, and (b) any 16 consecutive rows (a 16-lane phase
// with 64 banks, where rows of equal parity share a 128-byte bank half) use 8
// distinct positions per parity.
__device__ __forceinline__ int swz_key(int row) { return (row & 7) ^ ((row >> 3) & 1); }
__device__ __forceinline__ int swz(int row, int chunk) { return row * 128 + ((chunk ^ swz_key(row)) << 4); }

// 16 bytes per lane from a buffer straight into LDS: byte voff + soff of the
// buffer (voff per lane, soff wave-uniform) lands at lds_base + 16 l
// (lds_base wave-uniform, passed in m0). On the update tile's k loop this
// form issues at a markedly lower cost than global_load_lds_dwordx4 with a
// 64-bit address per lane; a load past the buffer's size returns zeros
// instead of faulting. Device pass only: the host pass of the single-source
// build just needs the kernel's stub.
//
// Issued through inline assembly: the compiler then does not track these LDS
// writes and puts no wait for them before later LDS reads (it cannot tell
// that those read the other stage). Completion is the caller's job: each
// k-slab is waited for by count (s_waitcnt vmcnt) before the block barrier
// that publishes it.
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 buffer_rsrc(const void *base, uint32_t bytes) {
  const uint64_t b = uint64_t(uintptr_t(base));
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane(int(uint32_t(b)));
  r[1] = __builtin_amdgcn_readfirstlane(int(uint32_t(b >> 32) & 0xffffu));   // stride 0
  r[2] = __builtin_amdgcn_readfirstlane(int(bytes));                        // size in bytes
  r[3] = 0x00020000;                                                         // raw 32-bit dwords
  return r;
}
__device__ __forceinline__ void buffer_load_lds16(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds_base) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds_base);
  const uint32_t so = __builtin_amdgcn_readfirstlane(soff);
  asm volatile("buffer_load_dwordx4 %1, %2, %3 offen lds" : : "{m0}"(m), "v"(voff), "s"(rsrc), "s"(so) : "memory");
#else
  (void)rsrc;
  (void)voff;
  (void)soff;
  (void)lds_base;
#endif
}
__device__ __forceinline__ void buffer_load_lds16(i32x4 rsrc, uint32_t voff, uint32_t soff, void *lds_base) {
  buffer_load_lds16(rsrc, voff, soff, uint32_t(uintptr_t(lds_base)));
}

// Transposing LDS read of 16-bit values (ds_read_b64_tr_b16). Within each
// group of 16 lanes, lane s gives the address of 4 consecutive values: row
// s / 4, columns 4 (s % 4) .. 4 (s % 4) + 3 of a 4 x 16 block; lane j then
// holds column j of the block, element i from row i.
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ half4 lds_read_tr16(const void *lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((__vector_size__(4 * sizeof(__fp16)))) __fp16 fp16x4;
  typedef __attribute__((address_space(3))) fp16x4 lds_fp16x4;
  const fp16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_fp16x4 *)(lds));
  return __builtin_bit_cast(half4, v);
#else
  (void)lds;
  return half4{};
#endif
}

// Byte offset of 16-byte chunk `chunk` of k-row `row`
// of a [k][n] operand stage (rows of `pitch` bytes). The key 4 (row & 3)
// spreads the 4 rows x 4 chunks that one half-wave reads with a transposing
// read (rows r..r+3 of a 16-row step, 64 bytes each) over all 64 banks.
__device__ __forceinline__ int kn_off(int row, int chunk, int pitch) {
  return row * pitch + ((chunk ^ ((row & 3) << 2)) << 4);
}

// Wait until every global -> LDS load this wave issued has landed (the
// compiler does not count them, see buffer_load_lds16); precedes the block barrier
// that publishes a stage.
__device__ __forceinline__ void lds_dma_wait() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#endif
}

// 8 consecutive iterate values as loaded, for a load issued ahead of its use.
struct XChunk {
  float4v a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = reinterpret_cast<const float4v *>(p)[0];
    b = reinterpret_cast<const float4v *>(p)[1];
  }
  __device__ __forceinline__ float get(int j) const { return j < 4 ? a[j] : b[j - 4]; }
};

// 8 consecutive values from global memory (16-byte aligned).
__device__ __forceinline__ void load8(const float *p, float (&v)[8]) {
  const float4v a = reinterpret_cast<const float4v *>(p)[0];
  const float4v b = reinterpret_cast<const float4v *>(p)[1];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = a[j];
    v[4 + j] = b[j];
  }
}

// As store8, marked non-temporal: the iterate written by an update is read
// only by the next launch, so its lines are not kept in this launch's L2,
// where they would evict operand panels that other tiles still read.
__device__ __forceinline__ void store8_stream(float *p, const float (&v)[8]) {
  float4v a, b;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    a[j] = v[j];
    b[j] = v[4 + j];
  }
  __builtin_nontemporal_store(a, reinterpret_cast<float4v *>(p));
  __builtin_nontemporal_store(b, reinterpret_cast<float4v *>(p) + 1);
}

template <typename T>
__device__ __forceinline__ void store8(T *p, const float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    half8 h;
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = _Float16(v[j]);
    *reinterpret_cast<half8 *>(p) = h;
  } else {
    float4v a, b;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = v[j];
      b[j] = v[4 + j];
    }
    reinterpret_cast<float4v *>(p)[0] = a;
    reinterpret_cast<float4v *>(p)[1] = b;
  }
}

// Elements j in [lo, hi) of 8 consecutive values (one vector store when all 8).
template <typename T>
__device__ __forceinline__ void store8_range(T *p, const float (&v)[8], int lo, int hi) {
  if (lo <= 0 && hi >= 8) {
    store8(p, v);
    return;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j >= lo && j < hi) p[j] = T(v[j]);
}

// Byte offset of 16-byte chunk `chunk` (0..7) of row `row` (0..31) of a
// wave's fp16 mirror block (32 rows of 64 values). The key spreads the rows
// that one transposing read touches (4 consecutive rows in each of four
// 8-row groups, 2 chunks each) over all 64 banks at two accesses per bank.
__device__ __forceinline__ int mir_off(int row, int chunk) {
  const int key = (((row >> 3) & 3) << 1) | ((row >> 1) & 1);
  return row * 128 + ((chunk ^ key) << 4);
}

// 8 fp16 values to p[lo .. hi) (all 8 with one 16-byte store when whole).
__device__ __forceinline__ void store_h8_range(_Float16 *p, const half8 &h, int lo, int hi) {
  if (lo <= 0 && hi >= 8) {
    *reinterpret_cast<half8 *>(p) = h;
    return;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j >= lo && j < hi) p[j] = h[j];
}

// The trace's partial over 8 consecutive columns of one row of an fp16 tile:
// sum of P (as stored) times X_0', four v_dot2_f32_f16 in column order with
// an fp32 running sum (each pair's products are formed exactly). The callers
// add these partials in fp64.
__device__ __forceinline__ float trace8(const half8 &p, const half8 &x0) {
  float f = 0.0f;
#pragma unroll
  for (int q = 0; q < 8; q += 2)
    f = __builtin_amdgcn_fdot2(half2v{p[q], p[q + 1]}, half2v{x0[q], x0[q + 1]}, f, false);
  return f;
}

template <int MODE, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void k_gemm(GemmArgs args) {
  using S = GemmShape<BM, BN, WGM, WGN>;
  typedef float T;
  constexpr int NT = S::kThreads;
  constexpr int V = Mfma::V;
  constexpr int BK = 8 * V;                      // k per slab (128-byte rows)
  constexpr int FM = S::FM, FN = S::FN, WTM = S::WTM, WTN = S::WTN;
  constexpr bool KN = (MODE == kUpdate || MODE == kLast);
  constexpr int QB = (BK / 4) * (BN / V) / NT;   // 4 x V blocks per thread, B slab (KN)
  static_assert(BM % (8 * S::kWaves) == 0 && BN % (8 * S::kWaves) == 0, "tile / wave mismatch");
  static_assert(!KN || QB * NT == (BK / 4) * (BN / V), "KN loader mismatch");
  static_assert(FM >= 1 && FN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "wave tile");
  typedef Mfma::frag frag;
  typedef T quad_t __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) char smem[S::kSmem];

  const Tile tile = args.tiles[blockIdx.x];
  if (tile.mat < 0) return;      // padding of the XCD-ordered list (whole block)
  // a Gram part (split K) covers k in [k0, k1) and stores its raw fp32 partial
  const bool part = MODE == kGram && tile.k1 > 0;
  // diagonal tile of a product of a matrix with itself (X X^T, A A; BM == BN):
  // the A and B operands are the same row panel, loaded once and read for both
  const bool diag = (MODE == kGram || MODE == kPoly) && BM == BN && tile.tm == tile.tn;
  const MatDesc d = args.mats[tile.mat];
  const int m0 = tile.tm * BM, n0 = tile.tn * BN;
  // X buffer offsets read from the table in memory (a run-time index into the
  // local copy of the descriptor would place that copy in scratch memory)
  T *Xc = reinterpret_cast<T *>(args.ws + args.mats[tile.mat].x[args.xin]);
  T *Xn = reinterpret_cast<T *>(args.ws + args.mats[tile.mat].x[args.xout]);
  T *Am = reinterpret_cast<T *>(args.ws + d.a);
  T *Bm = reinterpret_cast<T *>(args.ws + d.b);

  const T *Ap;
  const T *Bp;
  int lda, ldb, K;
  if (MODE == kGram) {                               // A = X X^T
    Ap = Xc; Bp = Xc; lda = ldb = d.Qp; K = d.Qp;
    if (part) {
      Ap += tile.k0;
      Bp += tile.k0;
      K = tile.k1 - tile.k0;
    }
  } else if (MODE == kPoly) {                        // A A
    Ap = Am; Bp = Am; lda = ldb = d.Pp; K = d.Pp;
  } else {                                           // B X or A X
    Ap = args.use_a ? Am : Bm; Bp = Xc; lda = d.Pp; ldb = d.Qp; K = d.Pp;
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lk = lane >> 5;
  const int wm = wave / WGN, wn = wave % WGN;

  // Direct global -> LDS loads (buffer_load_dwordx4 ... lds) of the K-major
  // operands: one wave instruction fills 8 consecutive LDS rows (1 KB) at the
  // wave-uniform base in m0, lane l landing at base + 16 l, i.e. row l / 8,
  // physical chunk l % 8; the lane therefore fetches logical chunk
  // (l % 8) ^ key(row). No registers, no ds_write instructions. Each operand
  // matrix is one buffer resource (under 2 GiB, the plan's limit); a lane's
  // byte offset is fixed for the tile, and the slab and the instruction's row
  // step (a multiple of the swizzle key's period) go into the scalar offset.
  const T *Abase = Ap, *Bbase = Bp;               // the operand matrices (Gram parts: from k0)
  const uint32_t abytes = uint32_t(d.Pp) * uint32_t(lda) * sizeof(T) - uint32_t(part ? tile.k0 : 0) * sizeof(T);
  const uint32_t bbytes = uint32_t(d.Pp) * uint32_t(ldb) * sizeof(T) - uint32_t(part ? tile.k0 : 0) * sizeof(T);
  // With 8 waves (two per SIMD) and two K-major operands (Gram, poly), only
  // the first 4 waves fetch, one per SIMD: the other wave of the SIMD keeps
  // the MFMA pipe busy while the fetching one waits to issue.
  constexpr int kFW = (S::kWaves == 8 && !KN) ? 4 : S::kWaves;
  constexpr uint32_t kRowStep = 8 * kFW;          // rows between a wave's instructions
  static_assert(kRowStep % 16 == 0 && BM % kRowStep == 0 && BN % kRowStep == 0, "swizzle period");
  auto dload = [&](int k0, int buf) {
    char *sA = smem + buf * S::kStage;
    char *sB = sA + BM * 128;
    const int rsub = lane >> 3, pch = lane & 7;
    if (wave >= kFW) return;
    {
      const i32x4 ra = buffer_rsrc(Abase, abytes);
      const int row = wave * 8 + rsub;
      const uint32_t voff = (uint32_t(m0 + row) * uint32_t(lda) + uint32_t((pch ^ swz_key(row)) * V)) * sizeof(T);
#pragma unroll
      for (int i = 0; i < BM / 8 / kFW; ++i)
        buffer_load_lds16(ra, voff, (uint32_t(k0) + uint32_t(i) * kRowStep * uint32_t(lda)) * sizeof(T),
                          sA + (wave + i * kFW) * 8 * 128);
    }
    if constexpr (!KN) {
      if (diag) return;                 // both operands are the same rows: one copy
      const i32x4 rb = buffer_rsrc(Bbase, bbytes);
      const int row = wave * 8 + rsub;
      const uint32_t voff = (uint32_t(n0 + row) * uint32_t(ldb) + uint32_t((pch ^ swz_key(row)) * V)) * sizeof(T);
#pragma unroll
      for (int i = 0; i < BN / 8 / kFW; ++i)
        buffer_load_lds16(rb, voff, (uint32_t(k0) + uint32_t(i) * kRowStep * uint32_t(ldb)) * sizeof(T),
                          sB + (wave + i * kFW) * 8 * 128);
    }
  };
  // the transposing loader of the [k][n] operand (update) into registers
  frag rk[KN ? 4 * QB : 1];
  auto kload = [&](int k0) {
    if constexpr (KN) {
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        const int q = tid + i * NT, kq = q % (BK / 4), nc = q / (BK / 4);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          rk[4 * i + r] = *reinterpret_cast<const frag *>(Bp + size_t(k0 + 4 * kq + r) * ldb + n0 + nc * V);
      }
    }
  };
  auto kstore = [&](int buf) {
    if constexpr (KN) {
      char *sB = smem + buf * S::kStage + BM * 128;
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        const int q = tid + i * NT, kq = q % (BK / 4), nc = q / (BK / 4);
        const int byte = 4 * kq * int(sizeof(T));
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const int n = nc * V + j;
          quad_t v;
          v[0] = rk[4 * i + 0][j];
          v[1] = rk[4 * i + 1][j];
          v[2] = rk[4 * i + 2][j];
          v[3] = rk[4 * i + 3][j];
          *reinterpret_cast<quad_t *>(sB + swz(n, byte >> 4) + (byte & 15)) = v;
        }
      }
    }
  };

  floatx16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // fragments of k-step s + 1 are read from LDS while the MFMAs of k-step s run
  auto compute = [&](int buf) {
    const char *sA = smem + buf * S::kStage;
    const char *sB = diag ? sA : sA + BM * 128;
    frag fa[2][FM], fb[2][FN];
    auto read = [&](int s, int slot) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[slot][i] = *reinterpret_cast<const frag *>(sA + swz(wm * WTM + i * 32 + lr, 2 * s + lk));
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        fb[slot][j] = *reinterpret_cast<const frag *>(sB + swz(wn * WTN + j * 32 + lr, 2 * s + lk));
      }
    };
    read(0, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (s < 3) read(s + 1, (s + 1) & 1);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) Mfma::mma(acc[i][j], fa[s & 1][i], fb[s & 1][j]);
    }
  };

  // K is a multiple of 128 (padding) and BK divides it. One LDS stage is
  // multiplied while the other is filled by direct loads (and the transposed
  // update operand) for the next slab.
  const int nk = K / BK;
  dload(0, 0);
  kload(0);
  kstore(0);
  lds_dma_wait();
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int nb = (kt + 1) & 1;
    if (kt + 1 < nk) {
      dload((kt + 1) * BK, nb);
      kload((kt + 1) * BK);
    }
    compute(kt & 1);
    if (kt + 1 < nk) kstore(nb);
    lds_dma_wait();
    __syncthreads();
  }

  // ------------------------------------------------------------ epilogue
  // acc[i][j][r] holds row 8 (r / 4) + 4 lk + r % 4 and column lr of MFMA tile
  // (i, j). Per 32-row block of the wave tile: stage in the wave's own LDS
  // area (fp32), then finish row-wise with 16-byte accesses, then (mirror
  // tiles) write the transpose column-wise. The waves do not wait for each
  // other during the epilogue.
  constexpr int P = S::kEpiPitch;
  constexpr int CG = WTN / 8;                     // 8-column groups per staged row
  float *ep = reinterpret_cast<float *>(smem + wave * S::kEpiWave);
  // per-matrix coefficients
  float alpha = args.alpha, beta = args.beta, gamma = args.gamma;
  if (args.kap) {
    const StepScale s = step_scale(args, tile.mat);
    if (MODE == kPoly) {
      alpha = float(double(args.alpha) * s.k2 * s.k2 * s.m);
      beta = float(double(args.beta) * s.k2 * s.m);
      gamma = float(double(args.gamma) * s.m);
    } else {
      alpha = float(double(args.alpha) * s.k2 * s.m);
      beta = float(double(args.beta) * s.m);
    }
  }
  // symmetric output and where it goes
  T *Sym = MODE == kGram ? Am : Bm;
  // Symmetric outputs are stored exactly symmetric: off-diagonal tiles also
  // store their transpose; a diagonal tile stores its upper triangle and the
  // transpose of it below the diagonal (its own lower triangle, computed with
  // a different rounding, is not used).
  const bool mirror = (MODE == kGram || MODE == kPoly) && !part;
  const bool dtile = mirror && tile.tm == tile.tn;
  double tsum = 0.0;

  // Poly: the A values of the b A term, loaded one 32-row block ahead (two register buffers). Task t of a lane:
  // row task / CG, 8 columns from (task % CG) 8 of the staged block.
  constexpr int NTASK = 32 * CG / 64;
  static_assert(NTASK * 64 == 32 * CG, "epilogue task split");
  // (the last step's X_0' is loaded where it is used: registers)
  constexpr bool APRE = MODE == kPoly;
  XChunk apre[APRE ? 2 : 1][NTASK];
  const T *asrc = MODE == kLast ? reinterpret_cast<const T *>(args.ws + d.x[0]) : Am;
  const int apitch = MODE == kLast ? d.Qp : d.Pp;
  auto aprefetch = [&](int i, int b) {
    const int grow0 = m0 + wm * WTM + i * 32, gcol0 = n0 + wn * WTN;
#pragma unroll
    for (int t = 0; t < NTASK; ++t) {
      const int task = lane + 64 * t;
      apre[b][t].load(asrc + size_t(grow0 + task / CG) * apitch + gcol0 + (task % CG) * 8);
    }
  };
  if constexpr (APRE) aprefetch(0, 0);

#pragma unroll
  for (int i = 0; i < FM; ++i) {
    if constexpr (APRE)
      if (i + 1 < FM) aprefetch(i + 1, (i + 1) & 1);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) ep[(8 * (r >> 2) + 4 * lk + (r & 3)) * P + j * 32 + lr] = acc[i][j][r];
    // the staging area is the wave's own and one wave's LDS operations are
    // performed in order: a wave-level barrier (no reordering) suffices
    __builtin_amdgcn_wave_barrier();
    const int grow0 = m0 + wm * WTM + i * 32, gcol0 = n0 + wn * WTN;
#pragma unroll
    for (int t = 0; t < NTASK; ++t) {
      const int task = lane + 64 * t;
      const int row = task / CG, cg = task % CG;
      float4v *e = reinterpret_cast<float4v *>(ep + row * P + cg * 8);
      float v[8];
      {
        const float4v e0 = e[0], e1 = e[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = e0[j];
          v[4 + j] = e1[j];
        }
      }
      const int grow = grow0 + row, gcol = gcol0 + cg * 8;
      if (MODE == kGram) {
        if (part) {
          store8(args.gpart + size_t(tile.slot) * (BM * BN) + size_t(grow - m0) * BN + (gcol - n0), v);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] *= alpha;
          store8_range(Sym + size_t(grow) * d.Pp + gcol, v, dtile ? grow - gcol : 0, 8);
        }
      } else if (MODE == kPoly) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          v[j] = beta * apre[i & 1][t].get(j) + alpha * v[j] + (grow == gcol + j ? gamma : 0.0f);
        const int lo = dtile ? grow - gcol : 0;
        store8_range(Sym + size_t(grow) * d.Pp + gcol, v, lo, 8);
      } else {
        if (args.fold) {
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] *= alpha;
        } else {
          float in[8];
          load8(Xc + size_t(grow) * d.Qp + gcol, in);
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] = beta * in[j] + alpha * v[j];
        }
        if (MODE == kUpdate || args.write_x) store8_stream(Xn + size_t(grow) * d.Qp + gcol, v);
        if (MODE == kLast) {
          // P as stored times X_0' (both in the iterate's scale): each product
          // exact in fp64
#pragma unroll
          for (int j = 0; j < 8; ++j) tsum += double(v[j]) * double(asrc[size_t(grow) * apitch + gcol + j]);
        }
      }
      if (mirror) {
        float4v e0, e1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          e0[j] = v[j];
          e1[j] = v[4 + j];
        }
        e[0] = e0;
        e[1] = e1;
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (mirror) {
      // transpose: output row = this tile's column, 8 consecutive source rows
#pragma unroll
      for (int t = 0; t < NTASK; ++t) {
        const int task = lane + 64 * t;
        const int rg = task & 3, col = task >> 2;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = ep[(rg * 8 + j) * P + col];
        const int orow = gcol0 + col, ocol = grow0 + rg * 8;
        const int hi = dtile ? orow - ocol : 8;         // strictly below the diagonal
        store8_range(Sym + size_t(orow) * d.Pp + ocol, v, 0, hi);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  if (MODE == kLast) {
    __syncthreads();                      // the block sum reuses wave 0's staging area
    const double r = block_sum<NT>(tsum, reinterpret_cast<double *>(smem));
    if (tid == 0) args.tpart[tile.slot] = r;
  }
}
