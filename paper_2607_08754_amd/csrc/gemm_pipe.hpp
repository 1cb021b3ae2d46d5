// Pipelined MFMA kernels of the Polar Express step on 16-bit MFMA operands,
// for both storage forms of the iterate (device code, included by kernels.hip
// after gemm.hpp, inside namespace slorr):
//
//   k_tile    one output tile per block, NS LDS stages (Gram, poly; update on
//             128-tiles)
//   k_short   a whole step of a set of short matrices
//   k_upd256  the persistent 256 x 256 update kernel
//
// Storage forms
//   _Float16  bf16 sets: scaled fp16 values.
//   Split     fp32 sets: every value x (scaled) is held as two fp16 numbers,
//             hi = fp16(x) and lo = fp16(x - hi), 4 bytes in all. Rows are
//             cut into runs of 32 values, 128 bytes each: 32 hi, then 32 lo.
//             hi + lo keeps 23 of fp32's 24 significand bits in the worst
//             case, and all of them for three values in four. A product of
//             two values is formed as lo hi + hi lo + hi hi, three fp16 MFMAs
//             with fp32 accumulation; the dropped lo lo is below 2^-22 of the
//             product. Both planes end at fp16's smallest number: values of X
//             below 2^-12 (in its scale: below 1) lose bits, down to 2^-36.
//
// Why the split: fp32 MFMA runs at 1/16 of the fp16 rate, so three fp16
// products cost 3/16 of one fp32 product, and per byte fetched or read from
// LDS a split slab feeds 1.5 times the MFMA work of a plain fp16 slab. Its
// error is no larger than fp32 MFMA's: a k-long sum is rounded once per 16
// values of k and term instead of once per 2 values, which outweighs the
// operands' last bit. Measured against 64 bits, fp32 MFMA / split: gradients
// 2.3e-6 / 1.5e-6 (200 x 260), 6.4e-6 / 4.1e-6 (512 x 2048), 5.0e-6 / 3.3e-6
// (ViT-B/16 in fp32); values 1e-7 both. Also nearer on spectra that one value
// dominates (300 times the rest: 3.2e-6 / 2.2e-6), of six decades (3.9e-5 /
// 2.6e-5), rows and columns of six decades, heavy tails, sparse, square and long
// matrices, T = 1 to 10. Further off where a row carries the norm and leaves the
// others at the smallest number: 1e3 times the rest 9.0e-7 / 5.8e-7, 1e5 times
// 2.5e-7 / 9.7e-6 (384 x 1536; the bar of fp32 sets is 1e-4); and by the operands'
// last bit on matrices of a few rows, whose sums are short (up to 16 rows, T = 6
// and 8: 1.1 to 3.0e-7 / 2.2 to 3.9e-7).
// One fp32 call, fp32 MFMA -> split: ViT-B/16 12.7 -> 4.7 ms, ViT-S (with the
// decoupled update) 2.41 -> 1.14 ms, ResNet-18 1.58 -> 0.71 ms, 4 matrices of
// 128 x 256 (T = 5) 250 -> 177 us.
//
// Call times "before -> after" in these files are pairs taken in turn on one
// machine for the step that the comment describes; machines differ by some
// percent and later steps shortened the same calls, so pairs do not add up.
#pragma once

struct Split {
  uint32_t bits;      // storage unit of one value; see the row layout above
};

template <typename T> struct Iter;
template <> struct Iter<_Float16> {
  static constexpr int kPlanes = 1, kBK = 64;      // k per 128-byte slab row
};
template <> struct Iter<Split> {
  static constexpr int kPlanes = 2, kBK = 32;
};

// Index of the 16-byte chunk that holds value `col` (a multiple of 4) of a
// row, and the byte of that chunk within a row of the matrix.
template <typename T>
__device__ __forceinline__ int chunk_of(int col, int plane) {
  if constexpr (Iter<T>::kPlanes == 1) return col >> 3;
  return (col >> 5) * 8 + plane * 4 + ((col & 31) >> 3);
}
template <typename T>
__device__ __forceinline__ size_t byte_of(size_t row, size_t ld, int col, int plane) {
  if constexpr (Iter<T>::kPlanes == 1) return (row * ld + size_t(col)) * 2;
  return (row * ld + size_t(col & ~31)) * 4 + size_t(plane * 64 + (col & 31) * 2);
}

// The planes of a scaled fp32 result, and the value they hold (exact in fp32:
// lo's last bit is never below the last bit of v).
template <typename T, int N, typename H>
__device__ __forceinline__ void to_planes(const float (&v)[N], H (&h)[Iter<T>::kPlanes]) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const _Float16 hi = _Float16(v[j]);
    h[0][j] = hi;
    if constexpr (Iter<T>::kPlanes == 2) h[Iter<T>::kPlanes - 1][j] = _Float16(v[j] - float(hi));
  }
}
template <typename T, typename H>
__device__ __forceinline__ float of_planes(const H (&h)[Iter<T>::kPlanes], int j) {
  float f = float(h[0][j]);
  if constexpr (Iter<T>::kPlanes == 2) f += float(h[Iter<T>::kPlanes - 1][j]);
  return f;
}

// The trace's partial over 8 consecutive columns: P (as stored) times X_0'.
// fp16: trace8; split: every product of the two held values exact in fp64.
template <typename T>
__device__ __forceinline__ double trace_planes(const half8 (&p)[Iter<T>::kPlanes], const half8 (&x0)[Iter<T>::kPlanes]) {
  if constexpr (Iter<T>::kPlanes == 1) return double(trace8(p[0], x0[0]));
  double t = 0.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) t += double(of_planes<T>(p, j)) * double(of_planes<T>(x0, j));
  return t;
}

// LDS byte offset of a shared array. The fetches below take offsets, not
// pointers: a generic pointer would be cast back to LDS with a null check.
__device__ __forceinline__ uint32_t lds_offset(const char *smem) {
#if defined(__HIP_DEVICE_COMPILE__)
  return uint32_t(uintptr_t((const __attribute__((address_space(3))) char *)smem));
#else
  (void)smem;
  return 0;
#endif
}

// s_waitcnt vmcnt(N), the other counters left alone (gfx9 encoding).
template <int N>
__device__ __forceinline__ void vm_wait() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Wait until at most `ahead` (<= A) slabs of fetches, L instructions each,
// issued by this wave are outstanding.
template <int L, int A>
__device__ __forceinline__ void vm_wait_slabs(int ahead) {
  if constexpr (A >= 2) {
    if (ahead >= 2) {
      vm_wait<2 * L>();
      return;
    }
  }
  if constexpr (A >= 1) {
    if (ahead >= 1) {
      vm_wait<L>();
      return;
    }
  }
  vm_wait<0>();
}

// The MFMAs of one 16-deep k step of a wave tile, operands swapped (the n
// operand first): acc[i][j][4 g + q] = C[row lr of 32-row block i][column
// 32 j + 8 g + 4 lk + q] of the wave tile. Split: the small cross terms
// first; successive MFMAs go to different accumulators.
template <typename T, int FM, int FN>
__device__ __forceinline__ void mma_step(floatx16 (&acc)[FM][FN], const half8 (&fa)[Iter<T>::kPlanes][FM],
                                         const half8 (&fb)[Iter<T>::kPlanes][FN]) {
  if constexpr (Iter<T>::kPlanes == 2) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[0][j], fa[Iter<T>::kPlanes - 1][i], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[Iter<T>::kPlanes - 1][j], fa[0][i], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[0][j], fa[0][i], acc[i][j], 0, 0, 0);
}

// One slab (128-byte rows): the fragments of k step s + 1 are read from LDS
// while the MFMAs of step s run. The A operand's rows start at wave row ar
// of sA; the n operand is K-major rows (KN = false, rows from br) or [k][n]
// rows of KNP bytes (columns from br), transposed on the read.
template <typename T, int FM, int FN, bool KN, int KNP>
__device__ __forceinline__ void compute_slab(floatx16 (&acc)[FM][FN], const char *sA, const char *sB, int ar, int br,
                                             int lane) {
  constexpr int PL = Iter<T>::kPlanes, KS = Iter<T>::kBK / 16;
  const int lr = lane & 31, lk = lane >> 5;
  half8 fa[2][PL][FM], fb[2][PL][FN];
  auto read = [&](int s, int slot) {
#pragma unroll
    for (int p = 0; p < PL; ++p) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[slot][p][i] = *reinterpret_cast<const half8 *>(sA + swz(ar + i * 32 + lr, 4 * p + 2 * s + lk));
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if constexpr (KN) {
          // lane L: k = 16 s + 8 (L / 32) + 0..7 of column n = L % 32 of the
          // fragment, as two transposing reads of 4 k-rows each
          const int g = lane >> 4, si = lane & 15;
          const int row = 16 * s + 8 * (g >> 1) + (si >> 2);
          const int col = br + j * 32 + 16 * (g & 1) + 4 * (si & 3);
          const int off = kn_off(row, chunk_of<T>(col, p), KNP) + 8 * (si & 1);
          const half4 lo = lds_read_tr16(sB + off);
          const half4 hi = lds_read_tr16(sB + off + 4 * KNP);
          fb[slot][p][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
          fb[slot][p][j] = *reinterpret_cast<const half8 *>(sB + swz(br + j * 32 + lr, 4 * p + 2 * s + lk));
        }
      }
    }
  };
  read(0, 0);
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    if (s + 1 < KS) read(s + 1, (s + 1) & 1);
    mma_step<T, FM, FN>(acc, fa[s & 1], fb[s & 1]);
  }
}

// ---------------------------------------------------------------------------
// One output tile per block, wave tiles of 64 columns, NS LDS stages: slab
// k + NS - 1 is fetched while slab k is multiplied; each slab is waited for
// by count (vector loads complete in issue order), then one block barrier
// publishes it and frees the stage of the slab before it. Launches of at most
// one block per CU take 4 stages (128 KB, which leaves one block per CU
// anyway): their tiles are bound by the latency of the slabs' fetches. Others
// take 2 stages and two blocks per CU. fp16, a set's call with a wait for all
// fetches right after each slab before, this after: ViT-Ti (48 matrices, 144
// Gram and poly tiles: 4 stages) 261 -> 242 us, ViT-S 565 -> 545, 24 odd shapes
// up to 1000 x 4100 707 -> 684.
template <typename T, int BM, int BN, int WGM, int WGN, int NS, int MODE>
struct TileShape {
  static constexpr int kWaves = WGM * WGN, kThreads = 64 * kWaves;
  static constexpr int WTM = BM / WGM, WTN = BN / WGN, FM = WTM / 32, FN = WTN / 32;
  static constexpr int PL = Iter<T>::kPlanes, BK = Iter<T>::kBK;
  static constexpr bool KN = MODE == kUpdate || MODE == kLast;
  static constexpr int KNP = BN * int(sizeof(T));          // bytes per k-row of a [k][n] stage
  static constexpr int kStageA = BM * 128, kStage = kStageA + BN * 128;
  static constexpr int kHalf = 32 * 128;                   // 32 rows x 64 fp16 of one plane
  static constexpr int kPitch = WTN + 4;                   // floats per row staged in fp32 (poly)
  static constexpr int kEpiWave = PL * kHalf + (MODE == kPoly ? 32 * kPitch * 4 : 0);
  // split symmetric products: the diagonal's sums of squares, behind the rest
  static constexpr bool kDiagSq = PL == 2 && (MODE == kGram || MODE == kPoly);
  static constexpr int kDiagOff = NS * kStage > kWaves * kEpiWave ? NS * kStage : kWaves * kEpiWave;
  static constexpr int kSmem = kDiagOff + (kDiagSq ? BM * 4 : 0);
  // with 8 waves (two per SIMD) and two K-major operands, the first 4 fetch
  static constexpr int kFW = (kWaves == 8 && !KN) ? 4 : kWaves;
  static constexpr int RPX = 1024 / KNP;                   // k-rows per [k][n] fetch
  static constexpr int kLoadsA = BM / 8 / kFW, kLoadsB = KN ? BK / RPX / kFW : BN / 8 / kFW;
  static_assert(WTN == 64 && WTM % 32 == 0 && BM == BN, "wave tile");
  static_assert(BM % (8 * kFW) == 0 && (8 * kFW) % 16 == 0, "swizzle period");
  static_assert(!KN || (RPX >= 1 && (RPX * kFW) % 4 == 0 && BK % (RPX * kFW) == 0), "kn_off key period");
  static_assert(!kDiagSq || kThreads == 2 * BM, "two threads per diagonal row");
  static_assert((NS - 2) * (kLoadsA + kLoadsB) < 64 && kSmem <= 160 * 1024, "vmcnt range, LDS");
};

template <typename T, int MODE, int BM, int BN, int WGM, int WGN, int NS>
__global__ __launch_bounds__(64 * WGM * WGN) void k_tile(GemmArgs args) {
  using S = TileShape<T, BM, BN, WGM, WGN, NS, MODE>;
  constexpr int PL = S::PL, BK = S::BK, FM = S::FM, FN = S::FN, WTM = S::WTM, WTN = S::WTN;
  constexpr int V = 16 / int(sizeof(T));            // storage units per 16 bytes
  constexpr bool SYM = MODE == kGram || MODE == kPoly;
  __shared__ __attribute__((aligned(16))) char smem[S::kSmem];

  const Tile tile = args.tiles[blockIdx.x];
  if (tile.mat < 0) return;      // padding of the XCD-ordered list (whole block)
  // a Gram part (split K) covers k in [k0, k1) and stores its raw fp32 partial
  const bool part = MODE == kGram && tile.k1 > 0;
  // diagonal tile of a product of a matrix with itself: one row panel, read
  // for both operands
  const bool diag = SYM && tile.tm == tile.tn;
  const MatDesc d = args.mats[tile.mat];
  const int m0 = tile.tm * BM, n0 = tile.tn * BN;
  // X buffer offsets read from the table in memory (a run-time index into the
  // local copy of the descriptor would place that copy in scratch memory)
  char *Xc = args.ws + args.mats[tile.mat].x[args.xin];
  char *Xn = args.ws + args.mats[tile.mat].x[args.xout];
  // (their order in memory is x[0], x[1], x[2], a, b: see MatDesc)
  char *Am = args.ws + d.a, *Bm = args.ws + d.b;
  const char *Ap, *Bp;
  int lda, ldb, K;
  if (MODE == kGram) {                               // A = X X^T
    Ap = Bp = Xc + (part ? size_t(tile.k0) * sizeof(T) : 0);
    lda = ldb = d.Qp;
    K = part ? tile.k1 - tile.k0 : d.Qp;
  } else if (MODE == kPoly) {                        // A A
    Ap = Bp = Am;
    lda = ldb = K = d.Pp;
  } else {                                           // B X or A X
    Ap = args.use_a ? Am : Bm;
    Bp = Xc;
    lda = K = d.Pp;
    ldb = d.Qp;
  }

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lk = lane >> 5;
  const int wm = wave / WGN, wn = wave % WGN;

  // Direct global -> LDS fetches: one buffer resource per
  // operand matrix, a fixed byte offset per lane, the slab and the row step
  // in the scalar offset.
  const uint32_t skip = part ? uint32_t(tile.k0) * uint32_t(sizeof(T)) : 0u;
  const uint32_t abytes = uint32_t(d.Pp) * uint32_t(lda) * uint32_t(sizeof(T)) - skip;
  const uint32_t bbytes = uint32_t(d.Pp) * uint32_t(ldb) * uint32_t(sizeof(T)) - skip;
  auto fetch_rows = [&](const char *base, uint32_t bytes, int ld, int row0, int k0, uint32_t dst) {
    const i32x4 rs = buffer_rsrc(base, bytes);
    const int row = wave * 8 + (lane >> 3);
    const uint32_t voff =
        (uint32_t(row0 + row) * uint32_t(ld) + uint32_t(((lane & 7) ^ swz_key(row)) * V)) * uint32_t(sizeof(T));
#pragma unroll
    for (int i = 0; i < BM / 8 / S::kFW; ++i)
      buffer_load_lds16(rs, voff, (uint32_t(k0) + uint32_t(i) * uint32_t(8 * S::kFW) * uint32_t(ld)) * uint32_t(sizeof(T)),
                        dst + (wave + i * S::kFW) * 1024);
  };
  const uint32_t lds0 = lds_offset(smem);
  auto dload = [&](int k0, int st) {
    if (wave >= S::kFW) return;
    const uint32_t sA = lds0 + uint32_t(st) * S::kStage, sB = sA + S::kStageA;
    fetch_rows(Ap, abytes, lda, m0, k0, sA);
    if constexpr (S::KN) {
      constexpr int CPR = S::KNP / 16;
      const i32x4 rb = buffer_rsrc(Bp, bbytes);
      const int row = wave * S::RPX + lane / CPR;
      const uint32_t voff = (uint32_t(row) * uint32_t(ldb) +
                             uint32_t(n0 + ((lane % CPR) ^ ((row & 3) << 2)) * V)) * uint32_t(sizeof(T));
#pragma unroll
      for (int i = 0; i < S::kLoadsB; ++i)
        buffer_load_lds16(rb, voff, (uint32_t(k0) + uint32_t(i * S::RPX * S::kFW)) * uint32_t(ldb) * uint32_t(sizeof(T)),
                          sB + (wave + i * S::kFW) * 1024);
    } else if (!diag) {
      fetch_rows(Bp, bbytes, ldb, n0, k0, sB);
    }
  };

  floatx16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // Split, diagonal tiles: the diagonal elements sum_k x_ik^2 are also formed
  // as fp32 sums of the whole values (two threads per row, half of a slab's k
  // each) and replace the MFMA's. Every term of such a sum is positive, so
  // what the MFMA drops adds up there and nowhere else: lo lo, and the bits
  // of the 8 products of a lane that lie below 2^-24 of the largest of them.
  // Measured as -9e-7 on the value of 128 x 256 sets after 5 steps (fp32 MFMA:
  // 1e-7), where the last polynomial is still steep.
  float dsq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  auto diag_slab = [&](const char *sA) {
    const int row = tid >> 1, half = tid & 1;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      half8 h[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) h[p] = *reinterpret_cast<const half8 *>(sA + swz(row, 4 * p + 2 * half + c));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = of_planes<Split>(h, j);
        dsq[j & 3] = fmaf(x, x, dsq[j & 3]);
      }
    }
  };

  // K is a multiple of 128 (padding) and BK divides it
  const int nk = K / BK;
#pragma unroll
  for (int q = 0; q < NS - 1; ++q)
    if (q < nk) dload(q * BK, q);
  for (int kt = 0, st = 0; kt < nk; ++kt, st = st + 1 == NS ? 0 : st + 1) {
    const int ahead = min(NS - 2, nk - 1 - kt);      // slabs fetched after slab kt so far
    if (diag) vm_wait_slabs<S::kLoadsA, NS - 2>(ahead);
    else vm_wait_slabs<S::kLoadsA + S::kLoadsB, NS - 2>(ahead);
    __syncthreads();                 // slab kt is published; slab kt - 1 is done
    if (kt + NS - 1 < nk) dload((kt + NS - 1) * BK, st == 0 ? NS - 1 : st - 1);
    const char *sA = smem + st * S::kStage;
    if (S::kDiagSq && diag) diag_slab(sA);
    compute_slab<T, FM, FN, S::KN, S::KNP>(acc, sA, diag ? sA : sA + S::kStageA, wm * WTM, wn * WTN, lane);
    // instruction order: the first k-step's fragment reads, then the MFMAs of
    // a step with the next step's reads spread among them (as in k_upd256).
    // ViT-Ti 234 -> 227 us a call, ViT-S in fp32 1092 -> 1077, ResNet-18 in fp32
    // 691 -> 682, LLM-560M 15.32 -> 15.20 ms; no set slower.
    constexpr int KS = BK / 16, kReads = PL * (FM + FN * (S::KN ? 2 : 1)), kMfma = (PL == 1 ? 1 : 3) * FM * FN;
    constexpr int kGroups = kReads < kMfma ? kReads : kMfma;
    __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);      // LDS reads
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int q = 0; q < kGroups; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, kMfma / kGroups, 0);        // MFMA
        if (s + 1 < KS) __builtin_amdgcn_sched_group_barrier(0x100, kReads / kGroups, 0);
      }
  }
  float *dsum = reinterpret_cast<float *>(smem + S::kDiagOff);
  if (S::kDiagSq && diag) {
    float v = (dsq[0] + dsq[1]) + (dsq[2] + dsq[3]);
    v += __shfl_xor(v, 1);
    if ((tid & 1) == 0) dsum[tid >> 1] = v;
  }
  __syncthreads();                   // the epilogue reuses the stages

  // ------------------------------------------------------------ epilogue
  // Per 32-row block of the wave tile, in the wave's own LDS area: 8-byte
  // writes of the fp16 planes from the accumulators, 16-byte reads of 8
  // consecutive columns for row-contiguous stores, transposing reads for the
  // mirror tile. One wave's LDS operations are performed in order, so a
  // wave-level barrier (no reordering) suffices between them. Poly stages its
  // fp32 sums first and finishes them where it has 8 consecutive columns of
  // A for the b A term.
  char *eh = smem + wave * S::kEpiWave;
  float *ef = reinterpret_cast<float *>(eh + PL * S::kHalf);
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
  // Symmetric outputs are stored exactly symmetric: off-diagonal tiles also
  // store their transpose; a diagonal tile stores its upper triangle and the
  // transpose of it below the diagonal.
  char *Sym = MODE == kGram ? Am : Bm;
  double tsum = 0.0;
  constexpr int NTASK = 32 * 8 / 64;                // 8-column pieces per lane and block
  // poly: A's values of the b A term; last: the X_0' values of the trace. A
  // block's are loaded together before its stores (in order of use the
  // compiler would wait for each behind the store before it), in fp16 a block
  // ahead: LLM-135M 2826 -> 2785 us a call, ViT-S 484 -> 480, in fp32 1145 -> 1136.
  constexpr bool kOld = MODE == kPoly || MODE == kLast;
  constexpr int kAhead = PL == 1 ? 1 : 0;
  half8 old[kOld ? 1 + kAhead : 1][NTASK][PL];
  auto old_load = [&](int i) {
    const char *src = MODE == kLast ? args.ws + d.x[0] : Ap;
    const size_t ld = MODE == kLast ? d.Qp : d.Pp;
#pragma unroll
    for (int t = 0; t < NTASK; ++t) {
      const int task = lane + 64 * t;
#pragma unroll
      for (int p = 0; p < PL; ++p)
        old[kAhead ? i & 1 : 0][t][p] = *reinterpret_cast<const half8 *>(
            src + byte_of<T>(size_t(m0 + wm * WTM + i * 32 + (task >> 3)), ld, n0 + wn * WTN + 8 * (task & 7), p));
    }
  };
  if constexpr (kOld && kAhead) old_load(0);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int grow0 = m0 + wm * WTM + i * 32, gcol0 = n0 + wn * WTN;
    if constexpr (kOld) {
      if (i + kAhead < FM) old_load(i + kAhead);
    }
    if (S::kDiagSq && diag) {
      const float dv = dsum[wm * WTM + i * 32 + lr];
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (grow0 + lr == gcol0 + 32 * j + 8 * g + 4 * lk + q) acc[i][j][4 * g + q] = dv;
    }
    if (part) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float4v f;
#pragma unroll
          for (int q = 0; q < 4; ++q) f[q] = acc[i][j][4 * g + q];
          *reinterpret_cast<float4v *>(args.gpart + size_t(tile.slot) * (BM * BN) + size_t(grow0 - m0 + lr) * BN +
                                       (gcol0 - n0) + 32 * j + 8 * g + 4 * lk) = f;
        }
      continue;
    }
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = acc[i][j][4 * g + q];
        if constexpr (MODE == kPoly) {
          *reinterpret_cast<float4v *>(ef + lr * S::kPitch + 32 * j + 8 * g + 4 * lk) = float4v{v[0], v[1], v[2], v[3]};
        } else {
          if (SYM || args.fold) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] *= alpha;
          } else {                                   // cubic step: the a X term
            half4 in[PL];
#pragma unroll
            for (int p = 0; p < PL; ++p)
              in[p] = *reinterpret_cast<const half4 *>(
                  Xc + byte_of<T>(size_t(grow0 + lr), d.Qp, gcol0 + 32 * j + 8 * g + 4 * lk, p));
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = beta * of_planes<T>(in, q) + alpha * v[q];
          }
          half4 h[PL];
          to_planes<T>(v, h);
#pragma unroll
          for (int p = 0; p < PL; ++p)
            *reinterpret_cast<half4 *>(eh + p * S::kHalf + mir_off(lr, 4 * j + g) + 8 * lk) = h[p];
        }
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < NTASK; ++t) {
      const int task = lane + 64 * t, row = task >> 3, cg = task & 7;
      const int grow = grow0 + row, gcol = gcol0 + 8 * cg;
      half8 h[PL];
      if constexpr (MODE == kPoly) {
        const half8 (&av)[PL] = old[kAhead ? i & 1 : 0][t];
        const float4v e0 = *reinterpret_cast<const float4v *>(ef + row * S::kPitch + 8 * cg);
        const float4v e1 = *reinterpret_cast<const float4v *>(ef + row * S::kPitch + 8 * cg + 4);
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          v[j] = fmaf(alpha, j < 4 ? e0[j & 3] : e1[j & 3], beta * of_planes<T>(av, j)) + (grow == gcol + j ? gamma : 0.0f);
        to_planes<T>(v, h);
#pragma unroll
        for (int p = 0; p < PL; ++p) *reinterpret_cast<half8 *>(eh + p * S::kHalf + mir_off(row, cg)) = h[p];
      } else {
#pragma unroll
        for (int p = 0; p < PL; ++p) h[p] = *reinterpret_cast<const half8 *>(eh + p * S::kHalf + mir_off(row, cg));
      }
      if constexpr (SYM) {
#pragma unroll
        for (int p = 0; p < PL; ++p)
          store_h8_range(reinterpret_cast<_Float16 *>(Sym + byte_of<T>(size_t(grow), d.Pp, gcol, p)), h[p],
                         diag ? grow - gcol : 0, 8);
      } else {
        if (MODE == kUpdate || args.write_x) {
#pragma unroll
          for (int p = 0; p < PL; ++p) {
            half8 *o = reinterpret_cast<half8 *>(Xn + byte_of<T>(size_t(grow), d.Qp, gcol, p));
            // a step's iterate is streamed out, X_T is read soon (k_upd256)
            if constexpr (MODE == kUpdate) __builtin_nontemporal_store(h[p], o);
            else *o = h[p];
          }
        }
        if constexpr (MODE == kLast) {
          tsum += trace_planes<T>(h, old[kAhead ? i & 1 : 0][t]);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    if constexpr (SYM) {
      // transpose: each 16-lane group takes 16 columns x 8 rows; two
      // transposing reads (rows 0-3, 4-7 of the group) leave lane s with
      // column 16 cb + s, rows 8 rg .. 8 rg + 7: one 16-byte row piece of
      // the mirror tile
#pragma unroll
      for (int t = 0; t < NTASK; ++t) {
        const int q = (lane >> 4) + 4 * t, rg = q & 3, cb = q >> 2, si = lane & 15;
        const int col = 16 * cb + 4 * (si & 3);            // this lane's 4-column piece
        const int r = 8 * rg + (si >> 2);
        const int off = (col & 7) * 2;                     // byte within the 16-byte chunk
        const int orow = gcol0 + 16 * cb + si, ocol = grow0 + 8 * rg;
#pragma unroll
        for (int p = 0; p < PL; ++p) {
          const char *e = eh + p * S::kHalf;
          const half4 lo = lds_read_tr16(e + mir_off(r, col >> 3) + off);
          const half4 hi = lds_read_tr16(e + mir_off(r + 4, col >> 3) + off);
          const half8 h = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          store_h8_range(reinterpret_cast<_Float16 *>(Sym + byte_of<T>(size_t(orow), d.Pp, ocol, p)), h, 0,
                         diag ? orow - ocol : 8);          // strictly below the diagonal
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  if constexpr (MODE == kLast) {
    __syncthreads();                      // the block sum reuses wave 0's staging area
    const double r = block_sum<S::kThreads>(tsum, reinterpret_cast<double *>(smem));
    if (tid == 0) args.tpart[tile.slot] = r;
  }
}

// ---------------------------------------------------------------------------
// Sets of short matrices (P <= 128, Q <= kMaxShortSlices slices of 128
// columns): one launch per step.
//
// Their products have one tile of rows, so that a launch per product holds a
// few blocks that start, wait for a tile's fetches and end: 25 launches for 4
// matrices of 128 x 256. Here a block owns one slice of 128 columns of X for a
// whole step, all of it in LDS: it adds the matrix's Gram partials (one per
// slice, from the launch before) to A, forms B (every block of the matrix does:
// 2 P^3, less than a launch), multiplies its slice, stores it in place and
// forms the slice's Gram partial for the next launch. The first launch forms
// X_0's partials.
//
// Blocks of 8 waves of 32 x 64. LDS: A, then B (rows of B, K-major slabs), and
// the slice, first as [k][n] rows (the update's operand), then as K-major rows
// (the Gram product's): 128 KB in split form, 64 KB in fp16.
// Partials are added in slice order. 4 matrices of 128 x 256, fp32, T = 5: 182
// -> 98 us a call; bf16, T = 6: 145 -> 74.
struct ShortArgs {
  GemmArgs g;                   // alpha, beta, gamma: poly's; xin, xout: the slice's buffers
  const float *pin;             // Gram partials read, 128 x 128 at each trace slot
  float *pout;                  // and written
  float gram_alpha, upd_alpha;
};
enum ShortStep { kShortFirst = 0, kShortStep = 1, kShortLast = 2 };

template <typename T, int STEP>
__global__ __launch_bounds__(512) void k_short(ShortArgs s) {
  constexpr int PL = Iter<T>::kPlanes, BK = Iter<T>::kBK, NSLAB = kTile / BK;
  constexpr int V = 16 / int(sizeof(T)), NT = 512, FN = 2;
  constexpr uint32_t ES = sizeof(T);
  constexpr int KNP = kTile * int(sizeof(T));        // bytes per k-row of the slice
  constexpr int kSlab = kTile * 128;                 // bytes per slab, either layout
  constexpr int kMat = NSLAB * kSlab;
  constexpr int NTASK = kTile * kTile / 8 / NT;      // 8-column pieces per thread
  static_assert(BK * KNP == kSlab, "slab sizes");
  __shared__ __attribute__((aligned(16))) char smem[2 * kMat + kTile * 4 + 64];
  char *sA = smem, *sX = smem + kMat;
  float *dsum = reinterpret_cast<float *>(smem + 2 * kMat);

  const Tile tile = s.g.tiles[blockIdx.x];
  if (tile.mat < 0) return;      // padding of the XCD-ordered list (whole block)
  const MatDesc d = s.g.mats[tile.mat];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lk = lane >> 5;
  const int wm = wave >> 1, wn = wave & 1;
  const int n0 = tile.tn * kTile;
  const char *Xc = s.g.ws + s.g.mats[tile.mat].x[s.g.xin];
  char *Xn = s.g.ws + s.g.mats[tile.mat].x[s.g.xout];

  // the slice, global -> LDS: 1 KB per wave instruction, kMat / 1024 in all
  {
    const i32x4 rs = buffer_rsrc(Xc, uint32_t(kTile) * uint32_t(d.Qp) * ES);
    const uint32_t lds0 = lds_offset(smem) + kMat;
#pragma unroll
    for (int i = 0; i < kMat / 1024 / 8; ++i) {
      const int q = wave + 8 * i;                    // 1 KB piece
      uint32_t voff;
      if constexpr (STEP == kShortFirst) {           // K-major: 8 rows of a slab
        const int slab = q / (kTile / 8), row = (q % (kTile / 8)) * 8 + (lane >> 3);
        voff = (uint32_t(row) * uint32_t(d.Qp) + uint32_t(n0 + slab * BK + ((lane & 7) ^ swz_key(row)) * V)) * ES;
      } else {                                       // [k][n]: 1024 / KNP k-rows
        constexpr int CPR = KNP / 16;
        const int row = q * (1024 / KNP) + lane / CPR;
        voff = (uint32_t(row) * uint32_t(d.Qp) + uint32_t(n0 + ((lane % CPR) ^ ((row & 3) << 2)) * V)) * ES;
      }
      buffer_load_lds16(rs, voff, 0u, lds0 + uint32_t(q) * 1024u);
    }
  }
  half8 x0[STEP == kShortLast ? NTASK : 1][PL];      // the trace's X_0' values
  if constexpr (STEP == kShortLast) {
#pragma unroll
    for (int k = 0; k < NTASK; ++k) {
      const int q = tid + k * NT;
#pragma unroll
      for (int p = 0; p < PL; ++p)
        x0[k][p] = *reinterpret_cast<const half8 *>(
            s.g.ws + d.x[0] + byte_of<T>(size_t(q / (kTile / 8)), d.Qp, n0 + (q % (kTile / 8)) * 8, p));
    }
  }
  // byte of 16-byte chunk (row, columns col .. col + 7, plane) of a K-major matrix in LDS
  auto at = [&](int row, int col, int plane) {
    return (col / BK) * kSlab + swz(row, PL == 1 ? (col % BK) >> 3 : plane * 4 + ((col % BK) >> 3));
  };
  // Split: the diagonal of X X^T as fp32 sums of squares of whole values (see
  // k_tile): four threads per row, a quarter of the columns each
  auto diag_sums = [&](const char *m) {
    if constexpr (PL == 2) {
      const int row = tid >> 2, part = tid & 3;
      float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        half8 h[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) h[p] = *reinterpret_cast<const half8 *>(m + at(row, 32 * part + 8 * c, p));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float x = of_planes<Split>(h, j);
          q[j & 3] = fmaf(x, x, q[j & 3]);
        }
      }
      float v = (q[0] + q[1]) + (q[2] + q[3]);
      v += __shfl_xor(v, 1);
      v += __shfl_xor(v, 2);
      if (part == 0) dsum[row] = v;
    }
  };
  floatx16 acc[1][FN];
  auto clear = [&]() {
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.0f;
  };
  const int row = wm * 32 + lr, colw = wn * 64 + 4 * lk;   // acc[0][j][4 g + q]: column colw + 32 j + 8 g + q
  auto fix_diag = [&]() {
    if constexpr (PL == 2) {
      const float dv = dsum[row];
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (row == colw + 32 * j + 8 * g + q) acc[0][j][4 * g + q] = dv;
    }
  };

  if constexpr (STEP != kShortFirst) {
    // A = alpha times the partials, 8 columns per thread and task; the loads of
    // all tasks of a partial are in flight together
    const float *src = s.pin + size_t(d.trace_begin) * (kTile * kTile);
    const int parts = d.trace_end - d.trace_begin;
    float4v sum[NTASK][2];
#pragma unroll
    for (int k = 0; k < NTASK; ++k) {
      const float4v *p = reinterpret_cast<const float4v *>(src) + 2 * (tid + k * NT);
      sum[k][0] = p[0];
      sum[k][1] = p[1];
    }
#pragma unroll 2
    for (int e = 1; e < parts; ++e) {
      float4v v[NTASK][2];
#pragma unroll
      for (int k = 0; k < NTASK; ++k) {
        const float4v *p = reinterpret_cast<const float4v *>(src + size_t(e) * (kTile * kTile)) + 2 * (tid + k * NT);
        v[k][0] = p[0];
        v[k][1] = p[1];
      }
#pragma unroll
      for (int k = 0; k < NTASK; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          sum[k][0][j] += v[k][0][j];
          sum[k][1][j] += v[k][1][j];
        }
    }
#pragma unroll
    for (int k = 0; k < NTASK; ++k) {
      const int q = tid + k * NT, r = q / (kTile / 8), c = (q % (kTile / 8)) * 8;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = s.gram_alpha * sum[k][j >> 2][j & 3];
      half8 h[PL];
      to_planes<T>(v, h);
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) *reinterpret_cast<half8 *>(sA + at(r, c, pl)) = h[pl];
    }
    __syncthreads();
    // B = a I + b A + c A A
    diag_sums(sA);
    clear();
#pragma unroll
    for (int b = 0; b < NSLAB; ++b)
      compute_slab<T, 1, FN, false, 0>(acc, sA + b * kSlab, sA + b * kSlab, wm * 32, wn * 64, lane);
    float alpha = s.g.alpha, beta = s.g.beta, gamma = s.g.gamma;
    if (s.g.kap) {
      const StepScale c = step_scale(s.g, tile.mat);
      alpha = float(double(s.g.alpha) * c.k2 * c.k2 * c.m);
      beta = float(double(s.g.beta) * c.k2 * c.m);
      gamma = float(double(s.g.gamma) * c.m);
    }
    if constexpr (PL == 2) __syncthreads();          // dsum
    fix_diag();
    half4 hb[FN][4][PL];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int col = colw + 32 * j + 8 * g;
        half4 a[PL];
#pragma unroll
        for (int p = 0; p < PL; ++p) a[p] = *reinterpret_cast<const half4 *>(sA + at(row, col, p) + ((col >> 2) & 1) * 8);
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          v[q] = fmaf(alpha, acc[0][j][4 * g + q], beta * of_planes<T>(a, q)) + (row == col + q ? gamma : 0.0f);
        to_planes<T>(v, hb[j][g]);
      }
    __syncthreads();                                 // every wave has read A
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int col = colw + 32 * j + 8 * g;
#pragma unroll
        for (int p = 0; p < PL; ++p)
          *reinterpret_cast<half4 *>(sA + at(row, col, p) + ((col >> 2) & 1) * 8) = hb[j][g][p];
      }
    vm_wait<0>();                                    // the slice's fetches
    __syncthreads();
    // X' = B X on the slice
    clear();
#pragma unroll
    for (int b = 0; b < NSLAB; ++b)
      compute_slab<T, 1, FN, true, KNP>(acc, sA + b * kSlab, sX + b * kSlab, wm * 32, wn * 64, lane);
    __syncthreads();                                 // every wave has read X
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int col = colw + 32 * j + 8 * g;
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = acc[0][j][4 * g + q] * s.upd_alpha;
        half4 h[PL];
        to_planes<T>(v, h);
#pragma unroll
        for (int p = 0; p < PL; ++p)
          *reinterpret_cast<half4 *>(sX + at(row, col, p) + ((col >> 2) & 1) * 8) = h[p];
      }
    __syncthreads();
    // the slice to memory, and the trace's partial
    double tsum = 0.0;
#pragma unroll
    for (int k = 0; k < NTASK; ++k) {
      const int q = tid + k * NT, r = q / (kTile / 8), c = (q % (kTile / 8)) * 8;
      half8 h[PL];
#pragma unroll
      for (int p = 0; p < PL; ++p) {
        h[p] = *reinterpret_cast<const half8 *>(sX + at(r, c, p));
        if (STEP == kShortStep || s.g.write_x)
          *reinterpret_cast<half8 *>(Xn + byte_of<T>(size_t(r), d.Qp, n0 + c, p)) = h[p];
      }
      if constexpr (STEP == kShortLast) tsum += trace_planes<T>(h, x0[k]);
    }
    if constexpr (STEP == kShortLast) {
      const double r = block_sum<NT>(tsum, reinterpret_cast<double *>(sA));   // B is done with
      if (tid == 0) s.g.tpart[tile.slot] = r;
    }
  } else {
    vm_wait<0>();
    __syncthreads();
  }
  if constexpr (STEP != kShortLast) {
    diag_sums(sX);
    clear();
#pragma unroll
    for (int b = 0; b < NSLAB; ++b)
      compute_slab<T, 1, FN, false, 0>(acc, sX + b * kSlab, sX + b * kSlab, wm * 32, wn * 64, lane);
    if constexpr (PL == 2) __syncthreads();
    fix_diag();
    float *out = s.pout + size_t(tile.slot) * (kTile * kTile) + size_t(row) * kTile + colw;
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4v f;
#pragma unroll
        for (int q = 0; q < 4; ++q) f[q] = acc[0][j][4 * g + q];
        *reinterpret_cast<float4v *>(out + 32 * j + 8 * g) = f;
      }
  }
}
// ---------------------------------------------------------------------------
// Update / Last on 256 x 256 tiles: a persistent kernel.
//
// One block per CU walks the launch's tile list with a stride of the grid
// size. The grid is a multiple of the XCD count, so every list entry runs on
// the XCD the list assigns it to, as in a launch of one block per tile.
//
// Tile contexts: at the start, lane t of every wave loads what tile t of the
// block's sequence needs (operand offsets, padded dims, tile coordinates) into
// a register table, read later with readlane. The main loop then issues no
// memory access besides the operand fetches, so a slab's wait counts only
// them (a descriptor load in the loop would need a wait that drains every
// fetch in flight). A block with more than 64 tiles reloads the table.
//
// Operand pipeline: k-slabs of BK in NS LDS stages, fetched NS - 1 slabs
// ahead. The slab sequence runs on across tiles: the first slabs of the next
// tile are fetched while the last ones of the current tile are multiplied and
// while its epilogue runs. A slab is waited for by count (s_waitcnt vmcnt
// with the fetches issued after it still outstanding; vector loads complete
// in issue order, and outstanding stores only make the wait longer), then one
// block barrier publishes it and frees the stage of the previous slab, into
// which the next fetch goes. LDS: the stages and a separate 32 KB epilogue
// staging area (4 KB per wave), 160 KB in all (one block per CU).
//
// The MFMA operands are swapped as in k_tile: the iterate panel is
// the instruction's first operand, so each lane's accumulator holds 4
// consecutive output columns of one row (acc[i][j][4 g + q] = C[row lr of
// 32-row block i][column 32 j + 8 g + 4 lk + q] of the wave tile). The
// epilogue scales and rounds them to fp16 and stages them with 8-byte LDS
// writes; 16-byte reads then give each lane 8 consecutive columns, 8 lanes
// per row, so the global stores write whole 128-byte row segments. Every
// output element is the same fp32 sum rounded once, as in k_tile.
//
// Edge tiles: the padded dims are multiples of 128, so a matrix whose dims are
// not multiples of 256 ends in tiles of which a half lies outside. The fetches
// stay inside the matrix, and the waves whose tile lies outside only fetch and
// keep the barriers.
template <typename T>
struct Upd256 {
  static constexpr int BM = 256, BN = 256, WGM = 2, WGN = 4, kWaves = 8, NT = 512;
  static constexpr int WTM = 128, WTN = 64, FM = 4, FN = 2;
  static constexpr int BK = Iter<T>::kBK;            // k per slab
  static constexpr int PL = Iter<T>::kPlanes;
  static constexpr int NS = 2;                       // LDS stages (fetch distance NS - 1)
  static constexpr int KAP = 128;                    // bytes per row of the B stage (K-major)
  static constexpr int KNP = BN * int(sizeof(T));    // bytes per k-row of the X stage
  static constexpr int kStageA = BM * KAP;
  static constexpr int kStage = kStageA + BK * KNP;
  static constexpr int kEpi = 32 * 128;              // per wave: 32 rows x 64 fp16
  static constexpr int kSmem = NS * kStage + kWaves * kEpi;
  // global -> LDS instructions per fetching wave and slab: B rows (8 rows of
  // 128 bytes each), X rows (1 KB each: 2 fp16 or 1 split k-row). Only the
  // first kFetchWaves waves fetch (one per SIMD): a wave stalls while its
  // fetches wait for the address unit, and the other wave of its SIMD keeps
  // the MFMA pipe busy meanwhile.
  static constexpr int kFetchWaves = 4;
  static constexpr int RPA = 1024 / KAP, RPX = 1024 / KNP;
  static constexpr int kLoadsA = BM / RPA / kFetchWaves, kLoadsX = BK / RPX / kFetchWaves;
  static constexpr int kLoads = kLoadsA + kLoadsX;
  static_assert(BK * sizeof(T) == 128, "128-byte slab rows");
  static_assert(NS >= 2 && kSmem <= 160 * 1024, "LDS per CU");
  static_assert((NS - 2) * kLoads < 64, "vmcnt range");
};

// Byte offset of 16-byte chunk `chunk` of row `row` of a wave's epilogue
// staging area (rows of 128 bytes). The key (row >> 1) & 7 gives the 16 rows
// of an 8-byte write's half-wave distinct (row parity, chunk) pairs, i.e.
// distinct bank pairs; a 16-byte read's 16-lane phase covers two rows whole.
__device__ __forceinline__ int epi_off(int row, int chunk) {
  return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4);
}

template <typename T, int MODE, bool FOLD>
__global__ __launch_bounds__(512) void k_upd256(GemmArgs args) {
  using U = Upd256<T>;
  constexpr int BK = U::BK, NS = U::NS, PL = U::PL;
  constexpr int V = 16 / int(sizeof(T));       // storage units per 16 bytes
  static_assert(MODE == kUpdate || MODE == kLast, "update kernels only");
  __shared__ __attribute__((aligned(16))) char smem[U::kSmem];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lk = lane >> 5;
  const int wm = wave / U::WGN, wn = wave % U::WGN;
  const int G = gridDim.x;
  // positions of this block's sequence: entry blockIdx.x + pos * G
  const int npos = args.ntiles > int(blockIdx.x) ? (args.ntiles - int(blockIdx.x) + G - 1) / G : 0;

  // register table of tile contexts, positions tb .. tb + 63 (lane t: tb + t)
  int tb = 0;
  int v_mat, v_tmn, v_slot, v_pq;
  uint32_t v_x;        // byte offset of the matrix's buffers / 256
  auto load_table = [&](int base) {
    tb = base;
    const int pos = base + lane;
    v_mat = -1;
    v_tmn = v_slot = v_pq = 0;
    v_x = 0;
    if (pos < npos) {
      const Tile t = args.tiles[int(blockIdx.x) + pos * G];
      v_mat = t.mat;
      if (t.mat >= 0) {
        const MatDesc *d = args.mats + t.mat;
        v_tmn = t.tm | t.tn << 8;      // tm < 64, tn < 4096 (the plan's size limits)
        v_slot = t.slot;
        v_pq = d->Pp / kTile | d->Qp / kTile << 8;   // Pp <= 16384, Qp <= 2^20
        v_x = uint32_t(d->x[0] >> 8);
      }
    }
  };
  struct Ctx {
    const char *Ap, *Bp;   // B (or A) rows, X rows
    char *Xn;              // output iterate
    const char *X0;        // X_0' (trace)
    int ldx, K, m0, n0, mat, slot;
  };
  // the first valid position >= pos (npos if none); reloads the table when
  // pos leaves it
  auto next_pos = [&](int pos) {
    for (; pos < npos; ++pos) {
      if (pos >= tb + 64) load_table(pos);
      if (__builtin_amdgcn_readlane(v_mat, pos - tb) >= 0) break;
    }
    return pos;
  };
  auto ctx_at = [&](int pos) {
    const int t = pos - tb;
    Ctx c;
    const int pq = __builtin_amdgcn_readlane(v_pq, t);
    c.ldx = (pq >> 8) * kTile;
    c.K = (pq & 255) * kTile;
    // a matrix's buffers follow each other: x[0], x[1], x[2], a, b (MatDesc)
    const size_t px = size_t(c.K) * c.ldx * sizeof(T), pa = size_t(c.K) * c.K * sizeof(T);
    char *base = args.ws + (size_t(uint32_t(__builtin_amdgcn_readlane(int(v_x), t))) << 8);
    c.X0 = base;
    c.Bp = base + size_t(args.xin) * px;
    c.Xn = base + size_t(args.xout) * px;
    c.Ap = base + 3 * px + (args.use_a ? 0 : pa);
    const int tmn = __builtin_amdgcn_readlane(v_tmn, t);
    c.m0 = (tmn & 255) * U::BM;
    c.n0 = (tmn >> 8) * U::BN;
    c.mat = __builtin_amdgcn_readlane(v_mat, t);
    c.slot = __builtin_amdgcn_readlane(v_slot, t);
    return c;
  };

  // global -> LDS fetch of slab k0 of tile c into stage st: B rows, K-major,
  // 8 rows of 128 bytes per wave instruction (lane l: row l / 8, physical
  // chunk l % 8, fetching the logical chunk the swizzle puts there); X rows
  // [k][n], 1 KB of k-rows per wave instruction in kn_off's layout. Through
  // buffer resources over the two operand matrices (the plan keeps every
  // matrix of these launches under 2 GiB): each lane's byte offset is fixed
  // for a tile, and the slab and the instruction's row step go into the
  // wave-uniform offset (successive instructions of a wave are a fixed number
  // of rows apart, and the swizzle key repeats over them).
  static_assert((U::kFetchWaves * U::RPA) % 16 == 0 && (U::kFetchWaves * U::RPX) % 4 == 0, "swizzle period");
  constexpr uint32_t ES = sizeof(T);
  const uint32_t lds0 = lds_offset(smem);
  auto dload = [&](const Ctx &c, int k0, int st) {
    if (wave >= U::kFetchWaves) return;
    const uint32_t sA = lds0 + uint32_t(st) * U::kStage, sB = sA + U::kStageA;
    {
      const i32x4 ra = buffer_rsrc(c.Ap, uint32_t(c.K) * uint32_t(c.K) * ES);     // K x K
      const int row = wave * U::RPA + (lane >> 3);
      const uint32_t voff = (uint32_t(c.m0 + row) * uint32_t(c.K) + uint32_t(((lane & 7) ^ swz_key(row)) * V)) * ES;
      const uint32_t step = uint32_t(U::kFetchWaves * U::RPA) * uint32_t(c.K) * ES;
#pragma unroll
      for (int i = 0; i < U::kLoadsA / 2; ++i)
        buffer_load_lds16(ra, voff, uint32_t(k0) * ES + uint32_t(i) * step, sA + (wave + i * U::kFetchWaves) * 1024);
      if (c.m0 + U::BM / 2 < c.K) {          // the lower half lies inside the matrix
#pragma unroll
        for (int i = U::kLoadsA / 2; i < U::kLoadsA; ++i)
          buffer_load_lds16(ra, voff, uint32_t(k0) * ES + uint32_t(i) * step, sA + (wave + i * U::kFetchWaves) * 1024);
      }
    }
    constexpr int CPR = U::KNP / 16;
    {
      const i32x4 rx = buffer_rsrc(c.Bp, uint32_t(c.K) * uint32_t(c.ldx) * ES);  // K x ldx
      const int row = wave * U::RPX + lane / CPR;
      int col = c.n0 + ((lane % CPR) ^ ((row & 3) << 2)) * V;
      col -= col >= c.ldx ? U::BN / 2 : 0;   // right half outside the matrix: the left half again, unused
      const uint32_t voff = (uint32_t(row) * uint32_t(c.ldx) + uint32_t(col)) * ES;
      const uint32_t step = uint32_t(U::kFetchWaves * U::RPX) * uint32_t(c.ldx) * ES;
#pragma unroll
      for (int i = 0; i < U::kLoadsX; ++i)
        buffer_load_lds16(rx, voff, uint32_t(k0) * uint32_t(c.ldx) * ES + uint32_t(i) * step,
                          sB + (wave + i * U::kFetchWaves) * 1024);
    }
  };

  floatx16 acc[U::FM][U::FN];
  auto compute = [&](int st) {
    const char *sA = smem + st * U::kStage;
    compute_slab<T, U::FM, U::FN, true, U::KNP>(acc, sA, sA + U::kStageA, wm * U::WTM, wn * U::WTN, lane);
    // instruction order: the first k-step's fragment reads, then the MFMAs
    // of a step with the next step's reads spread among them (one per MFMA;
    // split: two per three), so the reads land under the MFMAs instead of
    // bunching at the step's start
    constexpr int KS = BK / 16, kReads = PL * (U::FM + 2 * U::FN), kGroups = 8;
    constexpr int kMfma = (PL == 1 ? 1 : 3) * U::FM * U::FN;
    static_assert(kReads % kGroups == 0 && kMfma % kGroups == 0, "reads per MFMA");
    __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);      // LDS reads
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int q = 0; q < kGroups; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, kMfma / kGroups, 0);        // MFMA
        if (s + 1 < KS) __builtin_amdgcn_sched_group_barrier(0x100, kReads / kGroups, 0);
      }
  };

  load_table(0);
  int pos = next_pos(0);
  if (pos >= npos) return;
  Ctx cur = ctx_at(pos);

  // producer: the next slab to fetch (position ppos, context pc, slab pk);
  // nextc: the context of the tile after the consumer's
  static_assert(NS - 1 < kBigTile / BK, "the fetches run at most one tile ahead");
  int ppos = pos, pk = 0, npos_c = pos;   // npos_c: position of nextc
  Ctx pc = cur, nextc = cur;
  bool pvalid = true;
  int issued = 0;                      // slabs fetched so far
  auto produce = [&](int st) {
    if (!pvalid) return;
    dload(pc, pk * BK, st);
    ++issued;
    if (++pk == pc.K / BK) {
      ppos = next_pos(ppos + 1);
      pvalid = ppos < npos;
      if (pvalid) {
        pc = ctx_at(ppos);
        nextc = pc;
        npos_c = ppos;
      }
      pk = 0;
    }
  };
#pragma unroll
  for (int q = 0; q < NS - 1; ++q) produce(q);

  char *ep = smem + NS * U::kStage + wave * U::kEpi;
  // Last: the X_0' values of the trace, 8 consecutive columns per lane in
  // the epilogue's read-back layout, loaded two 32-row blocks ahead (cubic
  // steps: one; split: where they are used, the registers hold no more)
  constexpr int XB = PL == 2 ? 0 : FOLD ? 2 : 1;
  half8 x0v[MODE == kLast && XB ? XB : 1][4][PL];
  auto x0load = [&](const Ctx &c, int i) {
    if constexpr (MODE == kLast) {
      const int row_w = c.m0 + wm * U::WTM, col_w = c.n0 + wn * U::WTN;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int q = lane + 64 * t, row = q >> 3, ch = q & 7;
#pragma unroll
        for (int p = 0; p < PL; ++p)
          x0v[XB ? i % XB : 0][t][p] = __builtin_nontemporal_load(reinterpret_cast<const half8 *>(
              c.X0 + byte_of<T>(size_t(row_w + i * 32 + row), c.ldx, col_w + 8 * ch, p)));
      }
    }
  };
  int g = 0;                           // slab being multiplied (global count)
  for (;;) {
#pragma unroll
    for (int i = 0; i < U::FM; ++i)
#pragma unroll
      for (int j = 0; j < U::FN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    // K is a multiple of 128 (padding), so of BK
    const int nk = cur.K / BK;
    // a wave tile of an edge tile lies wholly inside the matrix or outside it
    const bool active = cur.m0 + wm * U::WTM < cur.K && cur.n0 + wn * U::WTN < cur.ldx;
    for (int kt = 0; kt < nk; ++kt, ++g) {
      vm_wait_slabs<U::kLoads, NS - 2>(issued - g - 1);   // slab g has landed (this wave's part)
      __syncthreads();                 // ... every wave's part; slab g - 1 is done
      produce((g + NS - 1) % NS);
      if (active) compute(g % NS);
    }

    // ---------------------------------------------------------- epilogue
    float alpha = args.alpha, beta = args.beta;
    if (args.kap) {                        // a cubic step's coefficients per matrix
      const StepScale s = step_scale(args, cur.mat);
      alpha = float(double(args.alpha) * s.k2 * s.m);
      beta = float(double(args.beta) * s.m);
    }
    const int row_w = cur.m0 + wm * U::WTM, col_w = cur.n0 + wn * U::WTN;
    double tsum = 0.0;
    if (active) {
#pragma unroll
      for (int i = 0; i < XB; ++i) x0load(cur, i);
#pragma unroll
      for (int i = 0; i < U::FM; ++i) {
        half4 hv[U::FN][4][PL];
#pragma unroll
        for (int j = 0; j < U::FN; ++j)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = acc[i][j][4 * q4 + q];
            if constexpr (FOLD) {
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] *= alpha;
            } else {
              half4 in[PL];
#pragma unroll
              for (int p = 0; p < PL; ++p)
                in[p] = *reinterpret_cast<const half4 *>(
                    cur.Bp + byte_of<T>(size_t(row_w + i * 32 + lr), cur.ldx, col_w + 32 * j + 8 * q4 + 4 * lk, p));
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] = beta * of_planes<T>(in, q) + alpha * v[q];
            }
            to_planes<T>(v, hv[j][q4]);
            *reinterpret_cast<half4 *>(ep + epi_off(lr, 4 * j + q4) + 8 * lk) = hv[j][q4][0];
          }
        // the staging area (one plane of the block) is the wave's own and one
        // wave's LDS operations are performed in order: a wave-level barrier
        // (no reordering) suffices
        __builtin_amdgcn_wave_barrier();
        if constexpr (MODE == kLast && XB == 0) x0load(cur, i);
        half8 hi[PL == 2 ? 4 : 1];
        if constexpr (PL == 2) {             // take the hi plane, then stage the lo plane
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int c = lane + 64 * t;
            hi[t] = *reinterpret_cast<const half8 *>(ep + epi_off(c >> 3, c & 7));
          }
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int j = 0; j < U::FN; ++j)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
              *reinterpret_cast<half4 *>(ep + epi_off(lr, 4 * j + q4) + 8 * lk) = hv[j][q4][PL - 1];
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = lane + 64 * t, row = c >> 3, ch = c & 7;
          half8 h[PL];
          h[PL - 1] = *reinterpret_cast<const half8 *>(ep + epi_off(row, ch));
          if constexpr (PL == 2) h[0] = hi[t];
#pragma unroll
          for (int p = 0; p < PL; ++p) {
            half8 *o = reinterpret_cast<half8 *>(cur.Xn + byte_of<T>(size_t(row_w + i * 32 + row), cur.ldx, col_w + 8 * ch, p));
            // the iterate of a step is streamed out (the next launch reads it,
            // and its lines would evict operand panels this launch still reads);
            // X_T, read by the gradient kernel two short launches later, is
            // stored normally (measured faster; split: always, a branch here
            // costs the registers that keep this kernel out of scratch memory)
            if constexpr (MODE == kUpdate) __builtin_nontemporal_store(h[p], o);
            else if (PL == 2 || args.write_x) *o = h[p];
          }
          if constexpr (MODE == kLast) {     // P as stored times X_0'
            tsum += trace_planes<T>(h, x0v[XB ? i % XB : 0][t]);
          }
        }
        if (XB && i + XB < U::FM) x0load(cur, i + XB);
        __builtin_amdgcn_wave_barrier();
      }
    }
    if constexpr (MODE == kLast) {
      // per-tile partial of the trace: waves in order, each a fixed butterfly
      const double w = wave_sum(tsum);
      if (lane == 0) *reinterpret_cast<double *>(ep) = w;
      __syncthreads();
      const double *ws8 = reinterpret_cast<const double *>(smem + NS * U::kStage);
      constexpr int kStep = U::kEpi / int(sizeof(double));
      if (!args.quads) {
        if (tid == 0) {
          double r = 0.0;
          for (int q = 0; q < U::kWaves; ++q) r += ws8[q * kStep];
          args.tpart[cur.slot] = r;
        }
      } else if (tid < 4) {                // quadrant (tid / 2, tid % 2): two waves
        const int qm = tid >> 1, qn = tid & 1, q = qm * U::WGN + 2 * qn;
        if (cur.m0 + qm * kTile < cur.K && cur.n0 + qn * kTile < cur.ldx)
          args.tpart[cur.slot + qn * (cur.K / kTile) + qm] = ws8[q * kStep] + ws8[(q + 1) * kStep];
      }
    }
    if (npos_c == pos) break;          // the fetches found no further tile
    pos = npos_c;
    cur = nextc;
  }
}
