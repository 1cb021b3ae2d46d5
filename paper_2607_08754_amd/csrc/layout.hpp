// Device-visible plan tables of the SLORR library (shared by host and kernels).
//
// Every matrix W_i (rows x cols, row-major) is iterated in its canonical "wide"
// orientation P x Q, P = min(rows, cols), Q = max(rows, cols); the canonical
// operand is W when rows <= cols and W^T otherwise (the short-side Gram product
// behind the 4 P^2 Q + 2 P^3 cost of Sec. 3). Canonical buffers are zero-padded
// to Pp x Qp (multiples of kTile) so that GEMM tiles never need bounds checks:
// zero rows/columns stay zero under X <- a X + (b XX^T + c (XX^T)^2) X.
#pragma once
#include <stdint.h>

namespace slorr {

constexpr int kTile = 128;       // padding granularity = the small GEMM block tile
constexpr int kBigTile = 256;    // the large GEMM block tile
constexpr int kSmallTile = 64;   // the GEMM block tile of launches with few tiles
constexpr int kPrepTile = 64;    // tile of the normalise / transpose kernel
constexpr int kChunk = 32768;    // elements per block of the decoupled-update kernel
constexpr int kThreads = 256;    // threads per block of the non-GEMM kernels
constexpr int kXcds = 8;         // XCDs of an MI355X; workgroup b runs on XCD b % 8
constexpr int kCus = 256;        // compute units of an MI355X
constexpr int kRedStripes = 8;   // split-K Gram reduce: blocks (row stripes) per tile

// Power-of-two operand scales of the fp16 iterate (bf16 weights) and of the
// split iterate (fp32 weights: two fp16 numbers per value). With the
// input normalised by ||W||_F every singular value of X stays <= u_t <= 2, so
// |X_ij| <= 2, |A_ij| <= 4 and |B_ij| <= max |b t + c t^2| over t in [0, 4]
// (< 9 for the default schedule); the scales keep these far below the fp16
// maximum (65504) while moving the typical entries (~1/sqrt(PQ)) well into
// the normal range.
constexpr float kScaleX16 = 4096.0f;
constexpr float kScaleA16 = 4096.0f;
constexpr float kScaleB16 = 1024.0f;

struct MatDesc {
  int32_t rows, cols;          // original shape
  int32_t P, Q, Pp, Qp;        // canonical and padded canonical shape
  int32_t tall;                // 1 if the canonical operand is W^T
  int32_t empty;               // rows == 0 or cols == 0
  int32_t norm_begin, norm_end;     // slots in the norm-partials array (canonical tiles)
  int32_t trace_begin, trace_end;   // slots in the trace-partials array
  int32_t pad0, pad1;
  uint64_t x[3];                    // byte offsets in the workspace: X_0 (kept for the
                                    // trace), then the iterates alternate in x[1], x[2].
                                    // x[0], x[1], x[2], a, b (quintic tables) follow each
                                    // other without gaps: k_upd256 keeps x[0] alone
  uint64_t a, b;
  uint64_t xt;                      // buffer holding X_T once the schedule has run
};

struct DynDesc {               // per call: caller pointers
  const void *w;
  void *g;                     // gradient buffer (fp32 or bf16)
};

struct CallParams {            // per call
  float *out_vals;
  const float *gscale;         // per-matrix upstream factors (device) or null
  float grad_scale;
  int32_t pad;
};

struct Tile {                  // one GEMM output tile / one prep tile / one Gram part
  int32_t mat, tm, tn, slot;   // mat < 0: padding entry, the block exits at once;
                               // slot: trace / norm / Gram-part partial of the tile
  int32_t k0, k1;              // Gram part: its k range [k0, k1); k1 = 0: all of K
  int32_t parts;               // Gram reduce entry: partials slot .. slot + parts - 1
  int32_t pad;
};

struct Chunk {                 // a contiguous run of a matrix's elements
  int32_t mat, begin, len, pad;
};

// Per matrix, written by the kernels. The iterate starts from X_0' = W / 2^e with
// 2^e the smallest power of two >= f + eps. The scaling rounds nothing; what X_0'
// then holds of W is up to the iterate's type: bf16 weights in fp16 and fp32
// weights in fp32 whole (fp16: down to 2^-36 of 2^e), the split form 23 or 24 bits
// of them, down to the same smallest value. The remaining factor
// kappa = 2^e / (f + eps), in [1, 2), is applied by the first step's
// coefficients: p_1(kappa x) = (a kappa) x + (b kappa^3) x^3 + (c kappa^5) x^5.
//
// The split iterate has a smallest value (2^-24 in its scale), so where eps is
// large against f its X_0' is W / 2^(e - h), with 2^(e - h) the smallest power
// of two >= f: X_0' has f's size, and X_0 = kappa 2^-h X_0'. Each step's iterate
// is held as 2^h_t X_t, h_t = max(0, h - g_t), g_t the steps' largest growth in
// powers of two so far (Plan::growth): as much of h as the bound on X_t allows,
// until the iterate has grown to its ordinary size. h = 0 where eps <= f's
// distance to the next power of two, and for the other iterates.
struct Scalars {
  double sumsq, f, feps, nhat, value;
  double s1, s2;               // gradient = g (s1 P - s2 W), P as it is held
  double kappa;                // 2^e / (f + eps); 0 when f + eps == 0
  double two_e;                // 2^(e - h): W = two_e X_0', so the trace sum(W * P)
                               // is two_e sum(X_0' * P) over the canonical buffers
  float pscale;                // W times pscale 2^pexp is X_0' in the iterate's scale
  int16_t pexp;                // (pexp > 0 where the product exceeds fp32's 2^127)
  int16_t shift;               // split iterate: h, see above
};

}  // namespace slorr
