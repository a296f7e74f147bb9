// Closed-form modulation dW = (G + lambda I)^-1 C for gfx950 (CDNA4).
//
// Operation (arXiv 2607.00712, Sec. 3.2, Eq. 5): one D x D SPD system with
// D_out right-hand sides, solved once at the end of warmup. The "inversion" is
// a Cholesky factorisation A = L L^T of A = G + lambda I followed by two
// triangular solves L Z = C and L^T dW = Z, all in fp32. Eq. 6's feasibility
// score follows from the same quantities: eps = s - <dW, C> - lambda ||dW||^2.
//
// Blocking: 64 x 64 blocks, nb = D / 64 block rows (ragged last block).
//
// Cholesky, one launch per panel (right-looking, the next panel fused in):
//   launch k (k = -1 .. nb-2) owns the trailing lower block triangle from
//   block k+1 on. Workgroups on the next panel column (r, k+1) apply the rank-64
//   update of panel k to their block and to the diagonal block A_{k+1,k+1} (each
//   its own copy in LDS), and run the rows of both through one elimination: the
//   diagonal block's rows become its factor and the block's rows
//   L_{r,k+1} = (A_{r,k+1} - L_{r,k} L_{k+1,k}^T) L_{k+1,k+1}^-T in the same
//   steps. All other workgroups apply A_rt -= L_rk L_tk^T. The diagonal blocks
//   themselves are never overwritten (other workgroups of the same launch read
//   them); their inverses (the identity run through the elimination by the
//   diagonal block's own workgroup) go to Dinv.
// The elimination is bound by its latency: 64 pivots, one after the other. It
//   runs in registers, a matrix row per lane, 16 columns at a time, the pivot row
//   reaching all lanes as a DPP broadcast inside the multiply-add (4 + 2 (15 - j)
//   instructions at step j); between the 16-column pieces the four waves apply
//   them as 16x16x4 MFMAs. A panel launch takes 10.5 us at the 1536-row solve
//   (15.5 with a factor and inverse by readlane, a product with the inverse and
//   loads behind a branch each): 1.5K cycles to issue the loads, 5.7K for their
//   latency, the cut and the products, four times 1.8K of elimination and 1.6K
//   of LDS traffic, updates and barriers.
// Triangular solves in block LDL^T form over 256-blocks (details below): the
//   inverses X_I of the 256 x 256 diagonal blocks of L and P_I = X_I^T X_I,
//   Lh = L diag(X_I) (stored transposed above the 256-block diagonal), then one right-looking
//   rank-256 GEMM launch per block for the forward and for the backward sweep,
//   with no diagonal work in them.
// The panel updates and the sweeps run on the bf16 matrix cores with every fp32
// operand cut into three bf16 parts (below); the other products are fp32 MFMA.
// Several layers at once (the end of warmup solves every layer): every kernel
// takes its layer from the last grid dimension and offsets its workspace
// pointers by the layers' workspace stride (dW by its own stride), so one
// launch per step covers all layers with each layer's arithmetic unchanged.
#include "ispa_internal.h"

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <utility>

namespace ispa {
namespace {

constexpr int kNb = 64;
constexpr int kSup = 4;  // panels per super-panel of the deferred trailing update
constexpr int kThreads = 256;

// Batched solves (one per layer, the layer from the last grid dimension): the
// layers' workspaces are `bytes` apart.
template <class T>
__device__ __forceinline__ T* at_layer(T* p, int64_t bytes, int layer) {
  return (T*)((char*)p + bytes * layer);
}

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// accumulator element r of lane l sits at (row, col) of the 32 x 32 quadrant
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

typedef unsigned int u32;
typedef float f32x2 __attribute__((ext_vector_type(2)));

// x[0..7] cut into three bf16 chunks of 8
__device__ __forceinline__ void split8(const float (&x)[8], u32x4 (&p)[3]) {
  // (-1, 0) and (0, -1) as packed bf16, kept out of the compiler's sight: as an
  // inline constant of a packed operand -1.0 is taken for the wrong half
  u32 lo = 0x0000bf80u, hi = 0xbf800000u;
  asm("" : "+s"(lo), "+s"(hi));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float a = x[2 * j], b = x[2 * j + 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const bf16x2 w = __builtin_convertvector((f32x2{a, b}), bf16x2);
      p[q][j] = __builtin_bit_cast(u32, w);
      if (q < 2) {  // what the part left: one multiply-add with the pair, exact
        a = __builtin_amdgcn_fdot2_f32_bf16(w, __builtin_bit_cast(bf16x2, lo), a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(w, __builtin_bit_cast(bf16x2, hi), b, false);
      }
    }
  }
}


// Wave-uniform wave index (a scalar, so that a wave's branch is a scalar branch).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// Rows 0 .. rows - 1 of a row-major matrix as a buffer: loads past them read zero
// and stores past them are dropped, without a branch around each. Offsets in
// bytes, per lane (kNoCol where its column is outside) plus a scalar one; the
// hardware tests their sum, also where the scalar one alone is past the end.
constexpr int kNoCol = (int)0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const float* base, int64_t ld, int rows) {
  int64_t nrec = rows > 0 ? rows * ld * 4 : 0;
  if (nrec > 0x7fffffff) nrec = 0x7fffffff;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)nrec, 0x00020000);
}
__device__ __forceinline__ float ld1(__amdgpu_buffer_rsrc_t rs, int off, int soff) {
  return __builtin_bit_cast(float, (u32)__builtin_amdgcn_raw_buffer_load_b32(rs, off, soff, 0));
}
__device__ __forceinline__ f32x4 ld4(__amdgpu_buffer_rsrc_t rs, int off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
}
__device__ __forceinline__ void st1(__amdgpu_buffer_rsrc_t rs, int off, int soff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(u32, v), rs, off, soff, 0);
}

// A 64 x 64 fp32 tile with 16-byte aligned rows: 16 rows of a column chunk fall
// into different banks both as 16-byte pieces (a row each) and as the 4-byte
// operands of a 16 x 16 product.
constexpr int kLd4 = 68;
typedef float RowTile[kNb][kLd4];

// 16 steps of elimination on the register rows of one wave. y: the 16 x 16
// pivot block, row l % 16 (symmetric, all 16 columns) in lane l, four copies;
// x: 16 columns of one matrix row per lane. At step j the pivot p = y[j] of
// lane j and its row s_c = y[c] reach every lane as DPP row broadcasts inside
// the multiply-adds, and
//   x[c] -= (x[j] / p) s_c,   y[c] -= (y[j] / p) s_c   (c > j).
// Lane j keeps p; at the end column j of x is divided by sqrt(p_j) (hardware square
// root and reciprocal, about 1 ulp each). Afterwards x holds the row times L^-T of the pivot block, a row of the
// factor L. Returns the lane's pivot: not positive where the block is not SPD.
// One asm block on fixed registers, so that the waits it needs are its own: a
// DPP operand is read at least two instructions after it is written, a
// reciprocal at least one after it is issued.
__device__ __forceinline__ float elim16(f32x16& y, f32x16& x) {
  float r, ny, nx, piv;
  unsigned long long lane_j = 0x0001000100010001ull;  // lane j of each row of 16
  asm volatile(
      "s_nop 1\n"
      "v_mov_b32 %[p], 0\n"
      ".set ej, 0\n"
      ".rept 16\n"
      ".if ej == 15\n"
      "s_nop 1\n"
      ".endif\n"
      "v_rcp_f32_dpp %[r], v[32+ej] row_newbcast:ej row_mask:0xf bank_mask:0xf\n"
      "v_cndmask_b32 %[p], %[p], v[32+ej], %[m]\n"
      "s_lshl_b64 %[m], %[m], 1\n"
      "v_mul_f32 %[nx], v[48+ej], -%[r]\n"
      "v_mul_f32 %[ny], v[32+ej], -%[r]\n"
      ".set ec, ej + 1\n"
      ".rept 15 - ej\n"
      "v_fmac_f32_dpp v[48+ec], v[32+ec], %[nx] row_newbcast:ej row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp v[32+ec], v[32+ec], %[ny] row_newbcast:ej row_mask:0xf bank_mask:0xf\n"
      ".set ec, ec + 1\n"
      ".endr\n"
      ".set ej, ej + 1\n"
      ".endr\n"
      "v_sqrt_f32 %[r], %[p]\n"
      "s_nop 1\n"
      "v_rcp_f32 %[r], %[r]\n"
      "s_nop 1\n"
      ".set ej, 0\n"
      ".rept 16\n"
      "v_mul_f32_dpp v[48+ej], %[r], v[48+ej] row_newbcast:ej row_mask:0xf bank_mask:0xf\n"
      ".set ej, ej + 1\n"
      ".endr\n"
      : "+{v[32:47]}"(y), "+{v[48:63]}"(x), [r] "=&v"(r), [ny] "=&v"(ny), [nx] "=&v"(nx), [p] "=&v"(piv),
        [m] "+s"(lane_j)
      :
      : "scc");
  return piv;
}

// D -= X_T X_S^T for up to two 16 x 16 pieces: D = T[16 i ..][16 c ..], X_T and X_S
// the rows 16 i of T and 16 c of S at columns 16 b. All reads are issued first.
struct Piece {
  RowTile* T;
  int i, c;
};
template <int N>
__device__ __forceinline__ void update16(const Piece (&p)[N], const RowTile& S, int b, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  float x[N][4], y[N][4], d[N][4];
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[u][k] = (*p[u].T)[16 * p[u].i + l16][16 * b + 4 * k + g];
      y[u][k] = S[16 * p[u].c + l16][16 * b + 4 * k + g];
      d[u][k] = (*p[u].T)[16 * p[u].i + 4 * g + k][16 * p[u].c + l16];
    }
  f32x4 acc[N] = {};
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int u = 0; u < N; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][k], y[u][k], acc[u], 0, 0, 0);
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) (*p[u].T)[16 * p[u].i + 4 * g + k][16 * p[u].c + l16] = d[u][k] - acc[u][k];
}

// Factor the 64 x 64 SPD block in S (lower part valid, its diagonal 16 x 16
// pieces symmetric) into L in place, and turn the 64 rows in Q into Q L^-T (the
// panel block's rows, or the identity, which becomes L^-T). All four waves
// call, after a barrier that follows the writes of S and Q. 16 columns at a
// time: waves 0 and 1 eliminate them in the rows of S and Q (each with its own
// copy of the pivot block), all waves then apply them to the next 16 columns,
// and waves 2 and 3 to the columns after those during the next elimination.
// Sets *bad on a non-positive pivot.
__device__ __forceinline__ void factor_rows(RowTile& S, RowTile& Q, int* bad) {
  const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll 1
  for (int b = 0; b < 4; ++b) {
    RowTile& T = wave == 0 ? S : Q;
    f32x16 y, x;
    if (wave < 2) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4 v = *(const f32x4*)&S[16 * b + (lane & 15)][16 * b + 4 * c];
        const f32x4 w = *(const f32x4*)&T[lane][16 * b + 4 * c];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          y[4 * c + j] = v[j];
          x[4 * c + j] = w[j];
        }
      }
    }
    __syncthreads();  // wave 1 holds the pivot block: wave 0 may overwrite it
    if (wave < 2) {
      const float piv = elim16(y, x);
      if (wave == 0 && !(piv > 0.f)) *bad = 1;
      const int own = wave == 0 ? lane - 16 * b : kNb;  // row of S from the pivot block on
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = own < 4 * c + j ? 0.f : x[4 * c + j];
        *(f32x4*)&T[lane][16 * b + 4 * c] = v;
      }
    } else if (b > 0) {
      // the last 16 columns' updates past the next ones
      for (int c = b + 1; c < 4; ++c) {
        for (int i = c + wave - 2; i < 4; i += 2) update16<1>({{&S, i, c}}, S, b - 1, lane);
        update16<2>({{&Q, wave - 2, c}, {&Q, wave, c}}, S, b - 1, lane);
      }
    }
    __syncthreads();
    if (b < 3) {
      // 3 - b pieces of S and 4 of Q, the first of S (the next pivot block) on wave 3
      const int c = b + 1;
      if (wave < 2 - b) {
        update16<2>({{&S, c + 1 + wave, c}, {&Q, wave, c}}, S, b, lane);
      } else if (wave < 3) {
        update16<1>({{&Q, wave, c}}, S, b, lane);
      } else {
        update16<2>({{&S, c, c}, {&Q, 3, c}}, S, b, lane);
      }
      __syncthreads();
    }
  }
}

// Panel products on the bf16 matrix cores (three-way cut operands): 64 rows x 32
// k of an operand are a half tile of three LDS planes of 64-byte rows, chunk c of
// row r at c ^ (r / 4 mod 4). Every place that applies a panel to a block sums
// its 64 k in the same order and subtracts the product on its own, so all forms
// of the factorisation give the same bits.
constexpr int kHalfTile = 64 * 64 * 3;  // bytes
struct Chunk {
  float v[8];
};
// 8 k of one row, at byte off
__device__ __forceinline__ void fetch8(Chunk& f, __amdgpu_buffer_rsrc_t rs, int off) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const f32x4 w = ld4(rs, off + 16 * q);
#pragma unroll
    for (int j = 0; j < 4; ++j) f.v[4 * q + j] = w[j];
  }
}
__device__ __forceinline__ int half_slot(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }
__device__ __forceinline__ void put8(char* half, const Chunk& f, int r, int c) {
  u32x4 p[3];
  split8(f.v, p);
#pragma unroll
  for (int q = 0; q < 3; ++q) *(u32x4*)(half + q * 4096 + half_slot(r, c)) = p[q];
}
__device__ __forceinline__ void read3(bf16x8 (&o)[3], const char* half, int r, int c) {
#pragma unroll
  for (int q = 0; q < 3; ++q) o[q] = *(const bf16x8*)(half + q * 4096 + half_slot(r, c));
}
// acc += A B^T over 16 k: the six products, the smallest first
__device__ __forceinline__ void mma6(f32x16& acc, const bf16x8 (&a)[3], const bf16x8 (&b)[3]) {
  constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
  for (int p = 0; p < 6; ++p) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa[p]], b[pb[p]], acc, 0, 0, 0);
}

__device__ __forceinline__ void tri_index(int t, int& ti, int& tj) {
  ti = (int)((sqrtf(8.f * t + 1.f) - 1.f) * 0.5f);
  while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
  while (ti * (ti + 1) / 2 > t) --ti;
  tj = t - ti * (ti + 1) / 2;
}

// L = lower(G) + lambda I with zeros above the diagonal up to the end of the
// row's 256-block (the part above the 256-block diagonal is never read before
// Lh^T is written there),
// status = 0. Row blockIdx.x, four columns per
// thread (n is a multiple of 4); only G's lower triangle is read.
__global__ void solve_init_kernel(const float* G, float* L, int n, float lambda, int* status, int64_t ws) {
  G = at_layer(G, ws, blockIdx.y);
  L = at_layer(L, ws, blockIdx.y);
  status = at_layer(status, ws, blockIdx.y);
  constexpr int kBlock = 256;  // the sweeps' block size
  const int r = blockIdx.x;
  const int end = min(n, (r / kBlock + 1) * kBlock);
  const float* g = G + (int64_t)r * n;
  float* l = L + (int64_t)r * n;
  for (int c = threadIdx.x * 4; c < end; c += blockDim.x * 4) {
    f32x4 v = c <= r ? *(const f32x4*)(g + c) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (c + j > r) v[j] = 0.f;
      else if (c + j == r) v[j] += lambda;
    }
    *(f32x4*)(l + c) = v;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *status = 0;
}

// Trailing update by the panels p0 .. p0 + NP - 1 of a 2 x 2 group of 64-blocks
// with top-left block (R, T), R >= T: A_rt -= L_rp L_tp^T for p in order, block
// (R + w / 2, T + w % 2) on wave w (blocks past the matrix, above the diagonal
// or in a column >= t_end are skipped). The four waves share L_rp (rows of
// blocks R, R + 1) and L_tp, cut and staged in LDS half a panel (32 k) at a time,
// loaded into registers two halves ahead; each wave's C block stays in registers
// from the first panel to the last, its loads under the first half's products.
// Each panel's product is subtracted on its own, in panel order, so the result
// is bit for bit that of one launch per panel. Half a panel takes about 3.7K
// cycles of a lone workgroup, 1.5K of them MFMAs (30 layers of 1536: the five
// deferred updates 461 us with fp32 MFMAs, 285 here).
template <int NP>
__device__ __forceinline__ void trailing_2x2(float* L, int n, int nblk, int p0, int R, int T, int t_end, char* lds) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int l32 = lane & 31, h = lane >> 5;
  const int br = R + (wave >> 1), bc = T + (wave & 1);
  const bool mine = br < nblk && bc <= br && bc < t_end;
  // half tile q: rows of block R, R + 1, T, T + 1; this thread's row and chunk
  const int row = threadIdx.x >> 2, chunk = threadIdx.x & 3;
  const int n4 = n * 4;
  const __amdgpu_buffer_rsrc_t rr = rows_rsrc(L + (int64_t)R * kNb * n, n, n - R * kNb);
  const __amdgpu_buffer_rsrc_t rt = rows_rsrc(L + (int64_t)T * kNb * n, n, n - T * kNb);
  Chunk f[2][4];  // the next two stages (the two halves of a panel)
  auto load = [&](Chunk (&f)[4], int s) {
    const int off = row * n4 + ((p0 + s / 2) * kNb + (s & 1) * 32 + chunk * 8) * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) fetch8(f[q], q < 2 ? rr : rt, off + (q & 1) * kNb * n4);
  };
  load(f[0], 0);
  load(f[1], 1);
  const __amdgpu_buffer_rsrc_t rb = rows_rsrc(L + (int64_t)br * kNb * n, n, n - br * kNb);
  int cof[2];  // column of block j of the accumulators, first row
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = bc * kNb + 32 * j + l32;
    cof[j] = col < n ? 4 * h * n4 + col * 4 : kNoCol;
  }
  float c[2][2][16];
  const char* const la = lds + (wave >> 1) * kHalfTile;
  const char* const lb = lds + (2 + (wave & 1)) * kHalfTile;
  f32x16 acc[2][2];
#pragma unroll 1
  for (int p = 0; p < NP; ++p) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (p + half > 0) __syncthreads();  // every wave is done with the previous stage
#pragma unroll
      for (int q = 0; q < 4; ++q) put8(lds + q * kHalfTile, f[half][q], row, chunk);
      if (p + 1 < NP) load(f[half], 2 * (p + 1) + half);
      __syncthreads();
      if (!mine) continue;
      if (p + half == 0) {  // the blocks themselves: needed after the panel's products
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) c[i][j][r] = ld1(rb, cof[j], (32 * i + acc_row(r, 0)) * n4);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        bf16x8 a[2][3], b[2][3];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          read3(a[i], la, 32 * i + l32, 2 * kk + h);
          read3(b[i], lb, 32 * i + l32, 2 * kk + h);
        }
        constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
        for (int pr = 0; pr < 6; ++pr)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][pa[pr]], b[j][pb[pr]], acc[i][j], 0, 0, 0);
      }
    }
    if (!mine) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[i][j][r] -= acc[i][j][r];
  }
  if (!mine) return;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) st1(rb, cof[j], (32 * i + acc_row(r, 0)) * n4, c[i][j][r]);
}

// The deferred update of a super-panel of kSup panels (p0 .. p0 + kSup - 1): the
// trailing triangle from block e on (rows r >= t >= e) in 2 x 2 groups.
__global__ __launch_bounds__(kThreads, 2) void chol_trail_kernel(float* L, int n, int p0, int e, int64_t ws) {
  __shared__ __attribute__((aligned(1024))) char lds[4 * kHalfTile];
  L = at_layer(L, ws, blockIdx.y);
  const int nblk = (n + kNb - 1) / kNb;
  int ti, tj;
  tri_index((int)blockIdx.x, ti, tj);
  trailing_2x2<kSup>(L, n, nblk, p0, e + 2 * ti, e + 2 * tj, nblk, lds);
}

// Panel-group updates that ride along in a single layer's panel launches (the
// look-ahead form of the factorisation), kLa panels at a time. Band b is block
// columns kLa b + 1 .. kLa b + kLa; task t applies the kLa panels of group
// sp[t] (panels kLa sp[t] ..) to every block of band band[t] at or below the
// diagonal, in groups[t] 2 x 2 groups, group column by group column. The
// tasks' workgroups follow the launch's `trail` groups.
constexpr int kLa = 2;
constexpr int kMaxTasks = 64;
struct CholExtra {
  int trail;  // -1: no tasks
  int n_tasks;
  int band[kMaxTasks], sp[kMaxTasks], groups[kMaxTasks];
};

// What workgroup wg of Cholesky launch k works on; the kernel and the host
// check of the look-ahead schedule share this decode. kind 0: the block of the
// next panel column in row R (column T = k + 1), which receives panel k when
// the launch applies it; kind 1: the 2 x 2 group of blocks with top-left
// (R, T), of which the blocks at or below the diagonal, inside the matrix and
// left of column t_end receive the np panels p0 ..; kind -1: nothing.
struct CholWork {
  int kind, R, T, p0, np, t_end;
};
__host__ __device__ inline CholWork chol_work_of(int wg, int nblk, int k, int t_end, const CholExtra& ex) {
  CholWork w = {-1, 0, 0, 0, 0, 0};
  const int m = nblk - 1 - k;  // panel-column workgroups of this launch
  if (ex.trail >= 0 && wg >= m + ex.trail) {
    int idx = wg - m - ex.trail;
    for (int t = 0; t < ex.n_tasks; ++t) {
      if (idx < ex.groups[t]) {
        const int e = ex.band[t] * kLa + 1, end = e + kLa < nblk ? e + kLa : nblk;
        for (int T = e; T < end; T += 2) {
          const int gr = (nblk - T + 1) / 2;  // groups of this group column
          if (idx < gr) {
            w = CholWork{1, T + 2 * idx, T, ex.sp[t] * kLa, kLa, end};
            return w;
          }
          idx -= gr;
        }
        return w;
      }
      idx -= ex.groups[t];
    }
    return w;
  }
  if (wg >= m) {
    const int rows = (nblk - k - 2 + 1) / 2;  // group rows of the trailing part
    int idx = wg - m, gj = 0;
    while (gj < rows && idx >= rows - gj) {
      idx -= rows - gj;
      ++gj;
    }
    if (gj < rows) w = CholWork{1, k + 2 + 2 * (gj + idx), k + 2 + 2 * gj, k, 1, t_end};
    return w;
  }
  w = CholWork{0, k + 1 + wg, k + 1, k, 1, 0};
  return w;
}

// Cholesky launch k (k = -1 .. nblk - 2): workgroups 0 .. m - 1 own the next
// panel column, blocks (k + 1 + i, k + 1), and (when `apply`) first subtract
// panel k from it; the others apply panel k to the trailing columns k + 2 ..
// t_end - 1 (all rows below) in 2 x 2 groups of blocks, group column by group
// column, then run the extra super-panel groups of `x` (none: x.trail = -1).
// Columns from t_end on receive panel k later, with the rest of its
// super-panel (chol_trail_kernel, or the extra groups of a later launch).
// Every workgroup of the panel column factors the diagonal block itself (no
// launch waits for another): the block's own rows ride through the same
// elimination, so L_rd needs no inverse and no product after it; the diagonal
// block's workgroup runs the identity through instead, which leaves the
// transposed inverse for Dinv.
__global__ __launch_bounds__(kThreads, 2) void chol_step_kernel(float* L, float* Dinv, int n, int k, int t_end,
                                                            int apply, int* status, int64_t ws, CholExtra ex) {
  // the panel's half tiles, then (in their place) the fp32 tiles S and Q
  __shared__ __attribute__((aligned(1024))) char lds[4 * kHalfTile];
  __shared__ int bad;
  L = at_layer(L, ws, blockIdx.y);
  Dinv = at_layer(Dinv, ws, blockIdx.y);
  status = at_layer(status, ws, blockIdx.y);
  const int nblk = (n + kNb - 1) / kNb;
  const CholWork wk = chol_work_of((int)blockIdx.x, nblk, k, t_end, ex);
  if (wk.kind < 0) return;
  if (wk.kind == 1) {
    if (wk.np == 1) {
      trailing_2x2<1>(L, n, nblk, wk.p0, wk.R, wk.T, wk.t_end, lds);
    } else {
      trailing_2x2<kLa>(L, n, nblk, wk.p0, wk.R, wk.T, wk.t_end, lds);
    }
    return;
  }
  apply = apply && k >= 0;
  RowTile &S = *(RowTile*)lds, &Q = *((RowTile*)lds + 1);
  static_assert(2 * sizeof(RowTile) <= sizeof(lds), "tiles");
  const int r = wk.R, d = k + 1;  // this workgroup's block row, the panel's column
  const int rr = min(kNb, n - r * kNb), nd = min(kNb, n - d * kNb);
  const bool off = r != d;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int r0 = (wave >> 1) * 32, c0 = (wave & 1) * 32;  // this wave's quadrant of S and Q
  if (threadIdx.x == 0) bad = 0;
  const int n4 = n * 4;
  const __amdgpu_buffer_rsrc_t rd = rows_rsrc(L + (int64_t)d * kNb * n, n, nd);
  const __amdgpu_buffer_rsrc_t rw = rows_rsrc(L + (int64_t)r * kNb * n, n, off ? rr : 0);
  Chunk fv[2], fu[2];
  const int row = threadIdx.x >> 2, chunk = threadIdx.x & 3;
  if (apply) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int o = row * n4 + (k * kNb + 32 * q + chunk * 8) * 4;
      fetch8(fv[q], rd, o);
      fetch8(fu[q], rw, o);
    }
  }
  // the quadrants in the accumulator layout; past the matrix S is the identity
  // (which keeps the factorisation defined) and Q zero
  float vs[16], vq[16];
  const int cof = c0 + l32 < nd ? (r0 + 4 * h) * n4 + (d * kNb + c0 + l32) * 4 : kNoCol;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    vs[e] = ld1(rd, cof, acc_row(e, 0) * n4);
    vq[e] = ld1(rw, cof, acc_row(e, 0) * n4);
  }
  if (apply) {
    // A_dd - L_dk L_dk^T and A_rd - L_rk L_dk^T
    char *lv = lds, *lu = lds + 2 * kHalfTile;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      put8(lv + q * kHalfTile, fv[q], row, chunk);
      put8(lu + q * kHalfTile, fu[q], row, chunk);
    }
    __syncthreads();
    f32x16 as = {}, aq = {};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8 a[3], b[3], u[3];
      read3(a, lv + (kk >> 1) * kHalfTile, r0 + l32, 2 * (kk & 1) + h);
      read3(b, lv + (kk >> 1) * kHalfTile, c0 + l32, 2 * (kk & 1) + h);
      read3(u, lu + (kk >> 1) * kHalfTile, r0 + l32, 2 * (kk & 1) + h);
      mma6(as, a, b);
      mma6(aq, u, b);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      vs[e] -= as[e];
      vq[e] -= aq[e];
    }
    __syncthreads();  // the half tiles are read
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = r0 + acc_row(e, lane), j = c0 + l32;
    const float one = i == j ? 1.f : 0.f;
    const float v = i < nd && j < nd ? vs[e] : one;
    if (i >= j) {  // the lower part, mirrored
      S[i][j] = v;
      S[j][i] = v;
    }
    Q[i][j] = off ? vq[e] : one;
  }
  __syncthreads();
  factor_rows(S, Q, &bad);
  if (off) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = threadIdx.x + q * kThreads;
      const int i = e >> 4, j = (e & 15) * 4;
      const f32x4 v = *(const f32x4*)&Q[i][j];
      const int o = j < nd ? i * n4 + (d * kNb + j) * 4 : kNoCol;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rw, o, 0, 0);
    }
    return;
  }
  float* D = Dinv + (int64_t)d * kNb * kNb;  // L^-1 = Q^T
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = threadIdx.x + q * kThreads;
    const int i = e >> 4, j = (e & 15) * 4;
    *(f32x4*)(D + i * kNb + j) = f32x4{Q[j][i], Q[j + 1][i], Q[j + 2][i], Q[j + 3][i]};
  }
  if (threadIdx.x == 0 && bad) atomicOr(status, 1);
}

// ---------------------------------------------------------------- 256-block
// Triangular solves in block LDL^T form. With 256 x 256 diagonal blocks L_II of
// L, X_I = L_II^-1, Lh_rI = L_rI X_I (unit block-lower Lh, L = Lh diag(L_II)) and
// P_I = X_I^T X_I (the inverse of the I-th diagonal block of the Schur
// complements):
//   L Z = C      <=>  Lh Y = C,  Z_I = X_I Y_I
//   L^T dW = Z   <=>  Lh^T dW = V,  V_I = P_I Y_I
// Both unit-triangular sweeps are right-looking rank-256 GEMM updates with no
// diagonal work, one launch per block: Y_r -= Lh_rI Y_I (r > I) and
// dW_I -= Lh_JI^T dW_J (I < J). Lh^T goes to the part of L above the 256-block
// diagonal (so its product with L_rI need not run in place), which both sweeps
// read: its rows as k in the forward sweep, as m in the backward one.
constexpr int kBb = 256;  // block size of the triangular sweeps

// X_I = L_II^-1 for 256-block I = blockIdx.x, 32-column strip blockIdx.y (in 64-block
// column b): X_bb = Dinv_b and, for a > b, X_ab = -Dinv_a sum_{c=b}^{a-1} L_ac X_cb
// (64-block indices inside the 256-block). Writes the full 256 x 32 strip of X_I
// (zeros above the diagonal and in 64-blocks past the end of the matrix).
// A chain of up to nine 64 x 64 x 32 products, bound by their latency and the fp32
// MFMAs (16 dependent steps of 16x16x4 each): 32-column strips for twice the
// workgroups of 64, the next factor tile loading into registers (as a buffer, no
// branch around a load) during each product. One layer of 1536
// 12.9 us, 30 layers 36.0 (64-column strips, each tile loaded when it is due: 21.4
// and 61.9).
constexpr int kXw = 32;   // columns of a strip
constexpr int kXld = 33;  // LDS row stride of its blocks
__global__ __launch_bounds__(kThreads) void inv256_kernel(const float* L, const float* Dinv, float* Xinv, int n,
                                                         int64_t ws) {
  __shared__ __attribute__((aligned(16))) RowTile U;
  __shared__ float Xc[4][kNb][kXld];
  L = at_layer(L, ws, blockIdx.z);
  Dinv = at_layer(Dinv, ws, blockIdx.z);
  Xinv = at_layer(Xinv, ws, blockIdx.z);
  const int nblk = (n + kNb - 1) / kNb;
  const int I = blockIdx.x, b = blockIdx.y >> 1, half = blockIdx.y & 1;
  const int g0 = I * 4;                 // first 64-block of the 256-block
  const int n64 = min(4, nblk - g0);    // 64-blocks inside the matrix
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int g = lane >> 4, l16 = lane & 15;
  const int tr = threadIdx.x >> 4, tc = (threadIdx.x & 15) * 4;  // a thread's piece of a 64 x 64 tile: rows tr + 16 q
  float* X = Xinv + (int64_t)I * kBb * kBb + b * kNb + half * kXw;  // the strip, rows of 256
  for (int a = 0; a < 4; ++a) {
    if (b < n64 && a >= b && a < n64) continue;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = threadIdx.x + q * kThreads;
      *(f32x4*)(X + (int64_t)(a * kNb + (e >> 3)) * kBb + (e & 7) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  if (b >= n64) return;

  f32x4 u[4];
  // tile (a, c) of the chain: L_ac, or Dinv_a for c = a
  auto issue = [&](int a, int c) {
    const bool dia = c == a;
    const float* src = dia ? Dinv + (int64_t)(g0 + a) * kNb * kNb
                           : L + (int64_t)(g0 + a) * kNb * n + (int64_t)(g0 + c) * kNb;
    const int ld = dia ? kNb : n, rows = dia ? kNb : min(kNb, n - (g0 + a) * kNb);
    const __amdgpu_buffer_rsrc_t rs = rows_rsrc(src, ld, rows);
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = ld4(rs, ((tr + 16 * q) * ld + tc) * 4);
  };
  // 64 x 32 product U Xb: wave w has rows 16 w .. 16 w + 15, two 16-column pieces
  auto product = [&](f32x4 (&acc)[2], const float (*Xb)[kXld]) {
#pragma unroll
    for (int k = 0; k < kNb; k += 4) {
      const float x = U[16 * wave + l16][k + g];
#pragma unroll
      for (int p = 0; p < 2; ++p)
        acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, Xb[k + g][16 * p + l16], acc[p], 0, 0, 0);
    }
  };
  auto keep = [&](int a, const f32x4 (&acc)[2]) {  // element r: row 4 g + r of the wave's 16
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int r = 0; r < 4; ++r) Xc[a][16 * wave + 4 * g + r][16 * p + l16] = acc[p][r];
  };

  const float* D = Dinv + (int64_t)(g0 + b) * kNb * kNb + half * kXw;
  f32x4 x0[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = threadIdx.x + q * kThreads;
    x0[q] = *(const f32x4*)(D + (e >> 3) * kNb + (e & 7) * 4);
  }
  if (b + 1 < n64) issue(b + 1, b);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = threadIdx.x + q * kThreads;
    const int r = e >> 3, c = (e & 7) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) Xc[b][r][c + j] = x0[q][j];
    *(f32x4*)(X + (int64_t)(b * kNb + r) * kBb + c) = x0[q];
  }
#pragma unroll 1
  for (int a = b + 1; a < n64; ++a) {
    f32x4 t[2] = {};
#pragma unroll 1
    for (int c = b; c <= a; ++c) {
      __syncthreads();  // U is read, and the block of X before this product is in LDS
#pragma unroll
      for (int q = 0; q < 4; ++q) *(f32x4*)&U[tr + 16 * q][tc] = u[q];
      if (c == a) keep(a, t);  // T goes through Xc[a]
      __syncthreads();
      if (c < a)
        issue(a, c + 1);
      else if (a + 1 < n64)
        issue(a + 1, b);
      if (c < a) product(t, Xc[c]);
    }
    f32x4 x[2] = {};
    product(x, Xc[a]);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      x[p] = -x[p];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        X[(int64_t)(a * kNb + 16 * wave + 4 * g + r) * kBb + 16 * p + l16] = x[p][r];
    }
    __syncthreads();  // every wave has read T
    keep(a, x);
  }
}

// P_I = X_I^T X_I for 256-block I = blockIdx.y, 64 x 64 tile blockIdx.x of its lower
// triangle, written with its mirror image. fp32 MFMA: on the cut operands these
// sums of squares came out low and scaled dW by 1.5e-7 (eps 3e-6 farther from 64
// bits). k starts at the tile's rows (X_I is lower triangular); 16 rows of
// both operands per step, two LDS buffers. (Six blocks of 30 layers 29 us, 72 with
// all tiles and all k; one layer 7.6 us, 14.6.)
constexpr int kXk = 16;
__global__ __launch_bounds__(kThreads) void xtx_kernel(const float* X, float* P, int d, int64_t ws) {
  __shared__ __attribute__((aligned(16))) float As[2][kXk][kNb + 32], Bs[2][kXk][kNb + 32];
  int ti, tj;
  tri_index((int)blockIdx.x, ti, tj);
  const int left = min(kBb, d - (int)blockIdx.y * kBb);
  const int end = (left + kNb - 1) / kNb * kNb;  // X_I is zero past the matrix
  if (ti * kNb >= end) return;
  X = at_layer(X, ws, blockIdx.z) + (int64_t)blockIdx.y * kBb * kBb;
  P = at_layer(P, ws, blockIdx.z) + (int64_t)blockIdx.y * kBb * kBb;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane >> 5, l32 = lane & 31;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int k = threadIdx.x >> 4, c = (threadIdx.x & 15) * 4;
  const float* xa = X + (int64_t)k * kBb + ti * kNb + c;
  const float* xb = X + (int64_t)k * kBb + tj * kNb + c;
  const int k0 = ti * kNb;
  f32x4 ra = *(const f32x4*)(xa + (int64_t)k0 * kBb), rb = *(const f32x4*)(xb + (int64_t)k0 * kBb);
  f32x16 acc = {};
  int buf = 0;
  for (int kk = k0; kk < end; kk += kXk, buf ^= 1) {
    *(f32x4*)&As[buf][k][c] = ra;
    *(f32x4*)&Bs[buf][k][c] = rb;
    if (kk + kXk < end) {
      ra = *(const f32x4*)(xa + (int64_t)(kk + kXk) * kBb);
      rb = *(const f32x4*)(xb + (int64_t)(kk + kXk) * kBb);
    }
    // one barrier per step: a wave that writes this buffer again has passed the next
    // step's barrier, which every wave reaches after reading this one
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kXk; j += 2) acc = mfma_f32(As[buf][j + h][wm + l32], Bs[buf][j + h][wn + l32], acc);
  }
  const int col = tj * kNb + wn + l32;
#pragma unroll
  for (int r = 0; r < 16; r += 4) {
    const int row = ti * kNb + wm + acc_row(r, lane);
    const f32x4 v = {acc[r], acc[r + 1], acc[r + 2], acc[r + 3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) P[(int64_t)(row + e) * kBb + col] = v[e];
    if (ti != tj) *(f32x4*)&P[(int64_t)col * kBb + row] = v;
  }
}

// <dW, C> and ||dW||^2 in two passes: each of kEpsBlocks workgroups reduces a
// grid-strided share (16-byte loads, n a multiple of 4) to one pair in
// part[2 * block], then a single workgroup adds the pairs into scalars[0], [1].
constexpr int kEpsBlocks = 512;
__device__ __forceinline__ void block_sum2(double& a, double& b, double (*red)[kThreads / 64]) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = a;
    red[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  a = 0;
  b = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    a += red[0][w];
    b += red[1][w];
  }
}
__global__ __launch_bounds__(kThreads) void eps_partial_kernel(const float* dw, const float* C, int64_t n,
                                                               double* part, int64_t ws, int64_t dws) {
  __shared__ double red[2][kThreads / 64];
  dw = at_layer(dw, dws, blockIdx.y);
  C = at_layer(C, ws, blockIdx.y);
  part = at_layer(part, ws, blockIdx.y);
  double a = 0, b = 0;
  const int64_t n4 = n / 4;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += (int64_t)gridDim.x * kThreads) {
    const f32x4 w = *(const f32x4*)(dw + 4 * i);
    const f32x4 c = *(const f32x4*)(C + 4 * i);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a += (double)w[j] * (double)c[j];
      b += (double)w[j] * (double)w[j];
    }
  }
  block_sum2(a, b, red);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = a;
    part[2 * blockIdx.x + 1] = b;
  }
}
// sc: [0] s = sum ||R||^2 (from the statistics), then written here: [2] <dW, C>,
// [3] ||dW||^2, [4] eps = s - <dW, C> - lambda ||dW||^2 (Eq. 6; each operation
// rounded on its own), [5] the status word as a double. eps_out / status_out,
// when given, receive eps and the status word as well.
__global__ __launch_bounds__(kThreads) void eps_final_kernel(const double* part, int n_part, double* sc,
                                                             double lambda, const int* status, double* eps_out,
                                                             int* status_out, int64_t ws) {
  __shared__ double red[2][kThreads / 64];
  const int layer = blockIdx.y;
  part = at_layer(part, ws, layer);
  sc = at_layer(sc, ws, layer);
  status = at_layer(status, ws, layer);
  double a = 0, b = 0;
  for (int i = threadIdx.x; i < n_part; i += kThreads) {
    a += part[2 * i];
    b += part[2 * i + 1];
  }
  block_sum2(a, b, red);
  if (threadIdx.x == 0) {
    const double e = __dsub_rn(__dsub_rn(sc[0], a), __dmul_rn(lambda, b));
    const int st = *status;
    sc[2] = a;
    sc[3] = b;
    sc[4] = e;
    sc[5] = (double)st;
    if (eps_out) eps_out[layer] = e;
    if (status_out) status_out[layer] = st;
  }
}

}  // namespace

namespace {

// ---------------------------------------------------------------- split GEMM
// The sweeps' GEMM, C(m, n) = [Cin(m, n) -] sum_k A(m, k) B(k, n), fp32 in and
// out, on the bf16 matrix cores: every operand value is cut into three bf16
// parts x = x0 + x1 + x2 (each the rounding of what is left: 3 x 8 significand
// bits hold fp32's 24 exactly), and of the nine products of two values the six
// with i + j <= 2 are summed in fp32; the three left out are below 2^-24 of the
// product (1.9 x 2^-25 found on values in [1, 1.02)), one fp32 rounding at most. Six
// bf16 MFMAs of 32x32x16 take 192 cycles where the fp32 form takes eight 32x32x2 of
// 64, and round the sum less often: each adds two groups of 8 products, a group
// rounded once, to nearest, after terms far below its largest are cut. The solve's
// dW on a given G and C, against 64 bits, with this and with fp32 MFMAs throughout:
// 6.3e-7 / 7.1e-7 at 1536, 9.0e-7 / 1.02e-6 at 5120; 0.42 to 0.96 times over sixty
// pairs of sizes from 128 to 5120 and rows centred, uncentred, of low rank plus
// noise, and of singular values spread over up to three orders, never above.
//
// Tile T x T (T = 64 Q), 4 waves of 32 Q x 32 Q, two or three workgroups on a CU.
// A thread holds one chunk of 8 k of one row of A and of B, loaded two stages
// ahead into registers and cut and written to LDS one stage ahead (two buffers,
// one barrier per stage): the cut is done once per workgroup, not per wave, and
// three planes of rows with k contiguous make an operand one ds_read_b128 per
// plane. A(m, k) = A[m lda + k] (A_KM = false) or A[k lda + m] (true), B likewise,
// so one copy of Lh serves both sweeps. The minuend's
// loads are issued before the last stage's products (30 layers of 1536: the
// first forward launch 275 us against 377 with the loads at the end, 395 with
// the fp32 kernel before). The stages run as straight code up to the last two,
// which lets the compiler place the cuts among the products (the batch 2.54 ->
// 2.43 ms; forcing an order of the instructions was 1-5% slower). What bounds it: 0.75 of the time of a launch is loads,
// cuts and barriers that two workgroups per CU do not hide (132 TFLOP/s there,
// 145 at one layer of 5120, against 92-110 before).
//
// The descriptor of a side ends at its last valid element, so k past K reads
// zero where k is the source's row and is masked where k is the column; rows and
// columns past M or N read zero. The order of an output's sum does not depend on
// the tile size: both give the same bits.
//
// bf16 has fp32's exponents, but the lower parts of a value need up to 16 more
// below: from 2^-110 down they lose bits (at 2^-126 a value would keep 8 of 24), and
// the largest fp32 values round to an infinite bf16. Tiles that hold such values,
// or whose sums leave fp32's range, are computed a second time with each row of both
// sides scaled by a power of two of its own. The test costs an or per pair of
// values and a barrier at the end (0.1-0.6% of a solve; scaling every operand up
// front 1.7-3%). An infinite or NaN value gives NaN.
struct SplitJob {
  const float* A;
  float* C;
  const float* Cin;  // minuend (null: C = A B)
  const float* B;
  int M, K;
  int64_t lda, ldc;
  int64_t la, lc;  // bytes per layer of A and of C / Cin
};
struct SplitArgs {
  SplitJob job[2];
  int n_jobs, N, layers;
  int64_t ldb, lb;  // lb: bytes per layer of B
  int tri = 0;     // A(m, k) is zero for k < m: skipped
  // one job over `batch` diagonal blocks: A, B and C advance by these elements per
  // block, and N is capped to what is left of the rows, N_left - kBb per block
  int batch = 1, N_left = 1 << 30;
  int64_t ba = 0, bb = 0, bc = 0;
};

// One side of the tile: T rows of the LDS planes (the m or n index), KS k; every
// thread holds one chunk of 8 k of one row. KM: k is the row of the source,
// else the column.
template <int T, bool KM>
struct SplitSide {
  static constexpr int kChunks = kThreads / T;  // per row
  static constexpr int kKs = 8 * kChunks;       // k per stage
  static constexpr int kBytes = T * kKs * 2 * 3;
  __amdgpu_buffer_rsrc_t rs;
  int voff[KM ? 8 : 1], step, k_first, dst;
  float v[8];
  u32 seen = 0;  // the first parts put so far, or-ed

  // byte of chunk c of row r in a plane: a 16-lane group of an operand read
  // (16 rows, one chunk) covers all banks once
  static __device__ __forceinline__ int slot(int r, int c) {
    return r * kKs * 2 + ((c ^ (kChunks == 4 ? (r >> 2) & 3 : (r >> 3) & 1)) << 4);
  }
  __device__ __forceinline__ void init(const float* src, int64_t ld, int i0, int iend, int K) {
    const int t = threadIdx.x;
    const float* base = KM ? src + i0 : src + (int64_t)i0 * ld;
    int64_t nrec = (KM ? (int64_t)(K - 1) * ld + (iend - i0) : (int64_t)(iend - i0 - 1) * ld + K) * 4;
    if (nrec > 0x7fffffff) nrec = 0x7fffffff;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)nrec, 0x00020000);
    const int ld4 = (int)(ld * 4);
    const int row = KM ? t % T : t / kChunks, chunk = KM ? t / T : t % kChunks;
    k_first = chunk * 8;
    dst = slot(row, chunk);
    if (KM) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        voff[k % (KM ? 8 : 1)] = row < iend - i0 ? (k_first + k) * ld4 + row * 4 : kNoCol;
      step = kKs * ld4;
    } else {
      voff[0] = row * ld4 + k_first * 4;
      step = kKs * 4;
    }
  }
  __device__ __forceinline__ void load(int s) {
    if (KM) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = __builtin_bit_cast(float, (u32)__builtin_amdgcn_raw_buffer_load_b32(rs, voff[k % (KM ? 8 : 1)], s * step, 0));
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4 w = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff[0] + q * 16, s * step, 0));
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * q + j] = w[j];
      }
    }
  }
  // k >= K of a stage reads the neighbouring columns of its row: zero them
  __device__ __forceinline__ void mask(int k0, int K) {
    if (KM) return;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k0 + k_first + k >= K) v[k] = 0.f;
  }
  __device__ __forceinline__ void put(char* lds) {
    u32x4 p[3];
    split8(v, p);
    seen |= p[0][0] | p[0][1] | p[0][2] | p[0][3];
#pragma unroll
    for (int q = 0; q < 3; ++q) *(u32x4*)(lds + q * (kBytes / 3) + dst) = p[q];
  }
  // every value put so far is below 2^-95, and not all are zero: a value below
  // 2^-110 beside a larger one loses at most 2^-39 of that one
  __device__ __forceinline__ bool tiny() const {
    const u32 exps = (seen | seen >> 16) & 0x7fff;
    return exps != 0 && (exps & 0x7000) == 0;
  }
  __device__ __forceinline__ float top() const {
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) m = fmaxf(m, fabsf(v[k]));
    return m;
  }
  __device__ __forceinline__ void scale(float by) {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] *= by;
  }
  // The power of two that brings the row's largest magnitude (top: of this thread's
  // chunk) to 2^50, so that sums of 2^9 products of two sides stay finite; the
  // rows' exponents go to exps. red: T x kChunks floats of LDS.
  __device__ __forceinline__ float row_scale(float top, float* red, int* exps) const {
    const int t = threadIdx.x;
    const int row = KM ? t % T : t / kChunks, chunk = KM ? t / T : t % kChunks;
    red[row * kChunks + chunk] = top;
    __syncthreads();
    for (int c = 0; c < kChunks; ++c) top = fmaxf(top, red[row * kChunks + c]);
    const int e = min(50 + 127 - (int)(__builtin_bit_cast(u32, top) >> 23), 64);
    exps[row] = e;
    return __builtin_amdgcn_ldexpf(1.f, e);
  }
};

template <int Q, bool A_KM, bool B_KM>
__global__ __launch_bounds__(kThreads, Q == 2 ? 2 : 3) void gemm_split_kernel(SplitArgs g) {
  constexpr int T = 64 * Q;
  using SideA = SplitSide<T, A_KM>;
  using SideB = SplitSide<T, B_KM>;
  constexpr int kKs = SideA::kKs, kSide = SideA::kBytes;
  __shared__ __attribute__((aligned(1024))) char smem[2][2 * kSide];
  __shared__ int exps[2][T], again;
  // consecutive tiles (n fastest, then m, job or block, layer) on one XCD
  const int idx = (int)(blockIdx.x & 7) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  auto tiles = [](int n) { return n > 0 ? (n + T - 1) / T : 0; };
  int per_layer = 0;
  for (int i = 0; i < g.batch; ++i)
    per_layer += tiles(g.job[0].M) * tiles(min(g.N, g.N_left - i * kBb));
  if (g.n_jobs > 1) per_layer += tiles(g.job[1].M) * tiles(g.N);
  if (idx >= per_layer * g.layers) return;
  const int layer = idx / per_layer;
  int t = idx - layer * per_layer, blk = 0;
  bool second = false;
  for (;;) {  // ends: t is below the sum of these counts
    const int n = tiles(g.job[0].M) * tiles(min(g.N, g.N_left - blk * kBb));
    if (t < n) break;
    t -= n;
    if (++blk == g.batch) {
      second = true;
      blk = 0;
      break;
    }
  }
  const SplitJob& jb = second ? g.job[1] : g.job[0];
  const int M = jb.M, K = jb.K;
  const int N = second ? g.N : min(g.N, g.N_left - blk * kBb);
  const int tiles_n = tiles(N);
  const int m0 = t / tiles_n * T, n0 = t % tiles_n * T;
  SideA sa;
  SideB sb;
  sa.init(at_layer(jb.A, jb.la, layer) + blk * g.ba, jb.lda, m0, M, K);
  sb.init(at_layer(jb.B, g.lb, layer) + blk * g.bb, g.ldb, n0, N, K);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int wm0 = (wave >> 1) * 32 * Q, wn0 = (wave & 1) * 32 * Q;

  f32x16 acc[Q][Q];
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j) acc[i][j] = f32x16{};

  float* C = at_layer(jb.C, jb.lc, layer) + blk * g.bc;
  const float* Cin = at_layer(jb.Cin, jb.lc, layer);  // never with several blocks

  // the minuend and the result: rows past M read zero and are not stored
  float cin[Q][Q][16];
  const __amdgpu_buffer_rsrc_t ro = rows_rsrc(C + (int64_t)m0 * jb.ldc, jb.ldc, M - m0);
  const __amdgpu_buffer_rsrc_t rc = rows_rsrc(Cin + (int64_t)m0 * jb.ldc, jb.ldc, jb.Cin != nullptr ? M - m0 : 0);
  const int ldc4 = (int)(jb.ldc * 4);
  int cof[Q];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int col = n0 + wn0 + 32 * j + l32;
    cof[j] = col < N ? (wm0 + 4 * h) * ldc4 + col * 4 : kNoCol;
  }

  const int steps = (K + kKs - 1) / kKs;
  const int s0 = g.tri ? m0 / kKs : 0;  // the first stage that is not all zero
  auto mask = [&](int s) {
    if ((s + 1) * kKs > K) {
      sa.mask(s * kKs, K);
      sb.mask(s * kKs, K);
    }
  };
  if (threadIdx.x == 0) again = 0;
  sa.load(s0);
  sb.load(s0);
  mask(s0);
  sa.put(smem[0]);
  sb.put(smem[0] + kSide);
  if (s0 + 1 < steps) {
    sa.load(s0 + 1);
    sb.load(s0 + 1);
  }
  __syncthreads();
  auto products = [&](const char* la) {
    const char* const lb = la + kSide;
#pragma unroll
    for (int kk = 0; kk < kKs / 16; ++kk) {
      bf16x8 a[Q][3], b[Q][3];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          a[i][q] = *(const bf16x8*)(la + q * (kSide / 3) + SideA::slot(wm0 + 32 * i + l32, 2 * kk + h));
          b[i][q] = *(const bf16x8*)(lb + q * (kSide / 3) + SideB::slot(wn0 + 32 * i + l32, 2 * kk + h));
        }
      }
      // the smallest products first
#pragma unroll
      for (int pr = 0; pr < 6; ++pr) {
        constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
          for (int j = 0; j < Q; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][pa[pr]], b[j][pb[pr]], acc[i][j], 0, 0, 0);
      }
    }
  };
  int s = s0;
  // stages whose next one is whole, in one piece of straight code: the next
  // stage's cuts between this one's matrix instructions (stages past the end
  // load zeros or unused neighbours)
  for (; (s + 2) * kKs <= K; ++s) {
    products(smem[(s - s0) & 1]);
    char* const next = smem[(s - s0 + 1) & 1];
    sa.put(next);
    sb.put(next + kSide);
    sa.load(s + 2);
    sb.load(s + 2);
    __syncthreads();
  }
  for (; s < steps; ++s) {
    const char* la = smem[(s - s0) & 1];
    if (s == steps - 1) {  // the minuend's loads pass under the last stage's products
#pragma unroll
      for (int i = 0; i < Q; ++i)
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            cin[i][j][r] = ld1(rc, cof[j], (32 * i + acc_row(r, 0)) * ldc4);
    }
    products(la);
    // the other buffer was read in stage s - 1, before the last barrier
    if (s + 1 < steps) {
      mask(s + 1);
      char* const next = smem[(s - s0 + 1) & 1];
      sa.put(next);
      sb.put(next + kSide);
      if (s + 2 < steps) {
        sa.load(s + 2);
        sb.load(s + 2);
      }
      __syncthreads();
    }
  }

  // Where a value or a sum left bf16's or fp32's range, or a thread's values were
  // all so small that their lower parts may have, the tile is computed again with
  // every row of both sides scaled by a power of two of its own.
  float odd = 0.f;  // NaN where a sum is not finite
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) odd = fmaf(acc[i][j][r], 0.f, odd);
  if (odd != 0.f || sa.tiny() || sb.tiny()) again = 1;
  __syncthreads();  // also: every wave has read the last stage
  if (__builtin_amdgcn_readfirstlane(again) != 0) {
    float ta = 0.f, tb = 0.f;
    for (int u = s0; u < steps; ++u) {
      sa.load(u);
      sb.load(u);
      mask(u);
      ta = fmaxf(ta, sa.top());
      tb = fmaxf(tb, sb.top());
    }
    const float ua = sa.row_scale(ta, (float*)smem[0], exps[0]);
    const float ub = sb.row_scale(tb, (float*)smem[1], exps[1]);
#pragma unroll
    for (int i = 0; i < Q; ++i)
#pragma unroll
      for (int j = 0; j < Q; ++j) acc[i][j] = f32x16{};
#pragma unroll 1
    for (int u = s0; u < steps; ++u) {
      sa.load(u);
      sb.load(u);
      mask(u);
      sa.scale(ua);
      sb.scale(ub);
      __syncthreads();
      sa.put(smem[0]);
      sb.put(smem[0] + kSide);
      __syncthreads();
      products(smem[0]);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i)
#pragma unroll
      for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          acc[i][j][r] = __builtin_amdgcn_ldexpf(
              acc[i][j][r], -(exps[0][wm0 + 32 * i + acc_row(r, lane)] + exps[1][wn0 + 32 * j + l32]));
  }

#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        st1(ro, cof[j], (32 * i + acc_row(r, 0)) * ldc4,
            jb.Cin != nullptr ? cin[i][j][r] - acc[i][j][r] : acc[i][j][r]);
}

}  // namespace

// Dinv: 64 x 64 inverses of the diagonal blocks of L, then X_I and P_I of the
// 256-blocks.
size_t solve_dinv_bytes(int d) {
  const int nblk = (d + kNb - 1) / kNb;
  const int nb = (d + kBb - 1) / kBb;
  return (size_t)nblk * kNb * kNb * sizeof(float) + 2 * (size_t)nb * kBb * kBb * sizeof(float);
}

namespace {

// Launches a split GEMM of up to two jobs for every layer: 128 x 128 tiles when
// there is at least one for each compute unit, else 64 x 64. 128 x 128 tiles
// halve the cutting and the operand reads per product (whole solves, 64 x 64
// throughout -> this rule: 30 layers of 1536 2.69 -> 2.43 ms, one of 5120 3.35 ->
// 3.12, 4096 2.00 -> 1.90, 3072 1.19 -> 1.17) but leave the chip idle with
// fewer (128 x 128 throughout: one layer of 1536 0.57 ms against 0.45, 2048 0.78
// against 0.63, four layers of 1536 0.72 against 0.67, one of 5120 3.21 against
// 3.12).
constexpr int kSplitBigTiles = 256;
template <bool A_KM, bool B_KM = true>
hipError_t launch_split(const SplitArgs& g, hipStream_t stream) {
  auto tiles = [&](int T) {
    auto up = [&](int n) -> int64_t { return n > 0 ? (n + T - 1) / T : 0; };
    int64_t n = 0;
    for (int i = 0; i < g.batch; ++i)
      n += up(g.job[0].M) * up(min(g.N, g.N_left - i * kBb));
    if (g.n_jobs > 1) n += up(g.job[1].M) * up(g.N);
    return n * g.layers;
  };
  const bool big = tiles(128) >= kSplitBigTiles;
  const int grid = (int)((tiles(big ? 128 : 64) + 7) / 8 * 8);
  if (grid == 0) return hipSuccess;
  if (big) {
    hipLaunchKernelGGL((gemm_split_kernel<2, A_KM, B_KM>), dim3(grid), dim3(kThreads), 0, stream, g);
  } else {
    hipLaunchKernelGGL((gemm_split_kernel<1, A_KM, B_KM>), dim3(grid), dim3(kThreads), 0, stream, g);
  }
  return hipGetLastError();
}

}  // namespace

// A second stream per device for one half of the sweeps' columns, with the
// events of the fork and the join (created once, kept for the process), from
// d = kSweepTwoFrom on; ISPA_SOLVE_TWO_STREAMS=0 / 1 switches it off / on at
// every size with at least two column tiles.
namespace {
constexpr int kSweepCols = 64;  // the halves split at a multiple of the tile width
constexpr int kSweepTwoFrom = 4096;  // smallest d whose sweeps go on two streams
struct SideStream {
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  bool tried = false;
};
std::mutex g_side_mu;
SideStream g_side[64];

SideStream* side_stream(int d) {
  const char* env = getenv("ISPA_SOLVE_TWO_STREAMS");
  if (env != nullptr ? env[0] != '1' : d < kSweepTwoFrom) return nullptr;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(g_side_mu);
  SideStream& t = g_side[dev];
  if (!t.tried) {
    t.tried = true;
    if (hipStreamCreateWithFlags(&t.s, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&t.fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&t.join, hipEventDisableTiming) != hipSuccess)
      t.s = nullptr;
  }
  return t.s != nullptr ? &t : nullptr;
}
}  // namespace

// The launches of a single layer's look-ahead factorisation (launch k at
// index k + 1): its workgroups, its t_end and its extra tasks (see launch_solve).
struct LookaheadPlan {
  std::vector<int> grid, t_end;
  std::vector<CholExtra> extra;
};
static void lookahead_plan(int nblk, int n_cu, LookaheadPlan* plan) {
  plan->grid.assign(nblk, 0);
  plan->t_end.assign(nblk, 0);
  plan->extra.assign(nblk, CholExtra{});
  int next_sp[kMaxTasks] = {};               // per band: the next group it receives
  const int n_bands = (nblk - 2) / kLa + 1;  // bands 1 .. n_bands - 1 start inside the matrix
  auto band_groups = [&](int b) {
    int g = 0;
    for (int T = b * kLa + 1; T < min(nblk, b * kLa + kLa + 1); T += 2) g += (nblk - T + 1) / 2;
    return g;
  };
  for (int k = -1; k <= nblk - 2; ++k) {
    const int m = nblk - 1 - k;
    const int t_end = k >= 0 ? min(nblk, k / kLa * kLa + kLa + 1) : 0;
    const int rows = (nblk - k - 2 + 1) / 2;
    const int cols = k >= 0 && t_end > k + 2 ? (t_end - k - 2 + 1) / 2 : 0;
    CholExtra x;
    memset(&x, 0, sizeof(x));
    x.trail = cols * rows - cols * (cols - 1) / 2;
    int cand[kMaxTasks][3], n_cand = 0;  // deadline, band, group
    for (int b = 1; b < n_bands; ++b) {
      const int sp = next_sp[b];
      if (sp <= b - 1 && k >= sp * kLa + kLa - 1) {
        cand[n_cand][0] = sp == b - 1 ? kLa * b - 1 : (kLa - 1) * b + sp;
        cand[n_cand][1] = b;
        cand[n_cand][2] = sp;
        ++n_cand;
      }
    }
    for (int i = 1; i < n_cand; ++i)  // by deadline, then band
      for (int j = i; j > 0 && (cand[j][0] < cand[j - 1][0] ||
                                (cand[j][0] == cand[j - 1][0] && cand[j][1] < cand[j - 1][1])); --j)
        for (int f = 0; f < 3; ++f) std::swap(cand[j][f], cand[j - 1][f]);
    // the rounds of workgroups the launch needs for its due tasks, filled up
    int used = m + x.trail, due = used;
    for (int i = 0; i < n_cand; ++i)
      if (cand[i][0] == k) due += band_groups(cand[i][1]);
    const int cap = (due + n_cu - 1) / n_cu * n_cu;
    for (int i = 0; i < n_cand; ++i) {
      const int b = cand[i][1];
      const int g = band_groups(b);
      if (cand[i][0] == k || used + g <= cap) {
        x.band[x.n_tasks] = b;
        x.sp[x.n_tasks] = cand[i][2];
        x.groups[x.n_tasks] = g;
        ++x.n_tasks;
        used += g;
        ++next_sp[b];
      }
    }
    plan->grid[k + 1] = used;
    plan->t_end[k + 1] = t_end;
    plan->extra[k + 1] = x;
  }
}

int solve_lookahead_check(int nblk, int n_cu) {
  if (nblk < 1 || (nblk - 2) / kLa + 1 >= kMaxTasks || n_cu < 1) return -1;
  LookaheadPlan plan;
  lookahead_plan(nblk, n_cu, &plan);
  // per block (r, c), r >= c: the next panel it must receive, and the last
  // launch that wrote it
  std::vector<int> next((size_t)nblk * nblk, 0), stamp((size_t)nblk * nblk, -2);
  for (int k = -1; k <= nblk - 2; ++k) {
    const int fail = k + 2;
    auto receive = [&](int r, int c, int p0, int np) {
      if (r < c || r >= nblk || c >= nblk) return false;
      const size_t b = (size_t)r * nblk + c;
      if (stamp[b] == k) return false;  // written twice in one launch
      stamp[b] = k;
      for (int p = p0; p < p0 + np; ++p) {
        // in panel order, panel p factored already (by launch p - 1), left of c
        if (p != next[b] || p > k || p >= c) return false;
        ++next[b];
      }
      return true;
    };
    for (int wg = 0; wg < plan.grid[k + 1]; ++wg) {
      const CholWork w = chol_work_of(wg, nblk, k, plan.t_end[k + 1], plan.extra[k + 1]);
      if (w.kind == 0) {
        if (!receive(w.R, w.T, k, k >= 0 ? 1 : 0)) return fail;
      } else if (w.kind == 1) {
        for (int i = 0; i < 4; ++i) {
          const int br = w.R + i / 2, bc = w.T + i % 2;
          if (br < nblk && bc <= br && bc < w.t_end && !receive(br, bc, w.p0, w.np)) return fail;
        }
      }
    }
    // the launch has factored column k + 1: every block of it complete
    for (int r = k + 1; r < nblk; ++r)
      if (next[(size_t)r * nblk + k + 1] != k + 1) return fail;
  }
  for (int r = 0; r < nblk; ++r)
    for (int c = 0; c <= r; ++c)
      if (next[(size_t)r * nblk + c] != c) return nblk + 1;
  return 0;
}

// A single layer's factorisation in the look-ahead form (below) from 48
// panels on (measured: 80 panels 3.38 -> 3.30 ms per solve, 24 panels 0.517 ->
// 0.526 ms); ISPA_SOLVE_LOOKAHEAD=0 / 1 switches
// it off / on at every size.
static bool solve_lookahead(int nblk) {
  if ((nblk - 2) / kLa + 1 >= kMaxTasks) return false;  // bands beyond the task table
  const char* env = getenv("ISPA_SOLVE_LOOKAHEAD");
  if (env != nullptr) return env[0] == '1';
  return nblk >= 48;
}

hipError_t launch_solve(const float* G, const float* C, int d, int d_out, float lambda, float* delta_w,
                        const SolveWork& w, hipStream_t stream) {
  const int nblk = (d + kNb - 1) / kNb;
  const int nb = (d + kBb - 1) / kBb;
  float* xinv = w.dinv + (size_t)nblk * kNb * kNb;  // [nb][256][256]
  float* pinv = xinv + (size_t)nb * kBb * kBb;       // [nb][256][256]
  float* L = w.L;
  float* Y = w.work;
  // layers: workspaces (G, C, L, Y, the inverses, status, scalars) `ws` bytes
  // apart, the layers' dW `dws` bytes apart
  const int nl = w.n_layers;
  const int64_t ws = w.ws_stride, dws = w.dw_stride;
  hipLaunchKernelGGL(solve_init_kernel, dim3(d, nl), dim3(256), 0, stream, G, L, d, lambda, w.status, ws);
  // Several layers: the panels are grouped kSup at a time (super-panels);
  // launch k applies panel k only to the columns of its own super-panel, and
  // the rest of the trailing triangle receives the super-panel's panels
  // together, in one launch that keeps each block in registers across them,
  // once its last panel is factored (a quarter of the trailing-matrix traffic
  // of applying each panel everywhere; the same arithmetic in the same order).
  // A single layer's factorisation is a chain of launches bound by their
  // latency, to which an extra launch per super-panel would add: it takes the
  // look-ahead form below from 48 panels on, and below that applies every
  // panel everywhere at once.
  const int sup = kSup;
  CholExtra none;
  memset(&none, 0, sizeof(none));
  none.trail = -1;
  if (nl == 1 && solve_lookahead(nblk)) {
    // Look-ahead form (one layer), with the panels in groups of kLa = 2: launch k
    // applies panel k only up to block column 2 s + 2, s = k / 2 its group (the
    // rest of the group and the first column of the next). The other columns
    // receive whole groups in tasks (band, group) that ride along as extra
    // workgroups in the panel launches: task (b, s) can run once panel 2 s + 1
    // is factored (launch 2 s + 1 on), after task (b, s - 1), and must be done
    // before launch 2 b applies panel 2 b to band b, so (b, b - 1) runs in
    // launch 2 b - 1 and (b, s < b - 1) by launch b + s. Each launch takes
    // every task whose deadline it is, then more of its available tasks,
    // earliest deadline first, as many as fill the rounds of workgroups on
    // the chip that the launch needs anyway (one at least). A task's
    // workgroup (two panels on a 2 x 2 group of blocks, ~15 us) takes longer
    // than the launch's panel chain (~10.5 us), so groups of more panels would
    // stretch the launches further; two rounds of workgroups per launch (two
    // fit on a compute unit) took 3.34 ms per solve at 80 panels, one round
    // 3.30. Each block still receives every panel once, in panel order, with the same
    // arithmetic: bit for bit the factor of the other forms.
    const int n_cu = attn_cu_count() > 0 ? attn_cu_count() : 256;
    LookaheadPlan plan;
    lookahead_plan(nblk, n_cu, &plan);
    for (int k = -1; k <= nblk - 2; ++k)
      hipLaunchKernelGGL(chol_step_kernel, dim3(plan.grid[k + 1], 1), dim3(kThreads), 0, stream, L, w.dinv, d, k,
                         plan.t_end[k + 1], k >= 0 ? 1 : 0, w.status, ws, plan.extra[k + 1]);
  } else {
    const int c_def = nl > 1 ? nblk + sup : 0;
    for (int k = -1; k <= nblk - 2; ++k) {
      const int c = k + 1;                          // the panel column this launch factors
      int apply = k >= 0 ? 1 : 0;
      int t_end;
      if (c > c_def) {
        t_end = nblk;
      } else if (c % sup == 0) {
        if (c > 0) {
          const int gr = (nblk - c + 1) / 2;
          hipLaunchKernelGGL(chol_trail_kernel, dim3(gr * (gr + 1) / 2, nl), dim3(kThreads), 0, stream, L, d,
                             c - sup, c, ws);
        }
        apply = 0;                                  // panel k reached column c with its super-panel
        t_end = c;                                  // and no column of its super-panel is left
      } else {
        t_end = min(nblk, (c / sup + 1) * sup);
      }
      const int m = nblk - 1 - k;                   // blocks of the next panel column
      const int rows = (nblk - k - 2 + 1) / 2;      // group rows of the trailing part
      const int cols = k >= 0 && t_end > k + 2 ? (t_end - k - 2 + 1) / 2 : 0;  // launch -1 has no panel to apply
      const int groups = cols * rows - cols * (cols - 1) / 2;
      hipLaunchKernelGGL(chol_step_kernel, dim3(m + groups, nl), dim3(kThreads), 0, stream, L, w.dinv, d, k, t_end,
                         apply, w.status, ws, none);
    }
  }
  // the inverses X_I of the diagonal blocks, P_I = X_I^T X_I, and Lh_rI = L_rI X_I
  // for the rows below, stored transposed above the diagonal blocks
  hipLaunchKernelGGL(inv256_kernel, dim3(nb, kBb / kXw, nl), dim3(kThreads), 0, stream, L, w.dinv, xinv, d, ws);
  hipLaunchKernelGGL(xtx_kernel, dim3(10, nb, nl), dim3(kThreads), 0, stream, xinv, pinv, d, ws);
  if (nb > 1) {
    // (m, n) = (column of block I, row below it), for every block that has rows below
    SplitArgs g = {};
    g.job[0] = SplitJob{xinv, L + kBb, nullptr, L + (int64_t)kBb * d, kBb, kBb, kBb, d, ws, ws};
    g.n_jobs = 1;
    g.N = g.N_left = d - kBb;
    g.layers = nl;
    g.ldb = d;
    g.lb = ws;
    g.tri = 1;
    g.batch = nb - 1;
    g.ba = (int64_t)kBb * kBb;
    g.bb = g.bc = (int64_t)kBb * d + kBb;
    const hipError_t e = launch_split<true, false>(g, stream);
    if (e != hipSuccess) return e;
  }
  // The sweeps treat each column of the right-hand side on its own, so from
  // d = 4096 on the columns go in two halves, each on a stream of its own (the
  // caller's and a second one), whose launches fill each other's last rounds
  // of tiles and hide each other's short launches; every element's arithmetic
  // is unchanged. Measured (one solve, alternating, medians of 5): d = 5120
  // 3.25 -> 3.11 ms, 4096 1.97 -> 1.89; d = 3072 1.17 -> 1.20, 2048 0.63 ->
  // 0.66, 1536 0.45 -> 0.49 ms (halves too small to fill the chip).
  auto yblk = [&](auto* base, int I) { return base + (int64_t)I * kBb * d_out; };
  auto kblk = [&](int I) { return min(kBb, d - I * kBb); };
  // Lh transposed: rows of block I, columns of block r > I
  auto up = [&](int I, int r) { return L + (int64_t)I * kBb * d + (int64_t)r * kBb; };
  auto sweeps = [&](int col0, int ncols, hipStream_t st) -> hipError_t {
    // forward sweep: Y_r -= Lh_rI Y_I (r > I) and dW_I = P_I Y_I. After the first
    // block the blocks go in pairs (I, I+1): one launch finishes Y_{I+1} and forms
    // dW_I, the next updates every later block with both (depth 512, so the
    // read-modify-write of the right-hand side below is shared by two blocks)
    // and forms dW_{I+1}. The A operand is Lh transposed, whose rows of blocks I
    // and I+1 are consecutive. Row pointers of
    // the right-hand side, Y and dW are taken at column 0 and moved to col0 here.
    auto fwd_launch = [&](const float* A, float* Ydst, const float* Ysrc, int M, const float* Bsum, int Ksum,
                          int P, const float* Bp, int Kp) -> hipError_t {
      SplitArgs g = {};
      int j = 0;
      if (M > 0) g.job[j++] = SplitJob{A, Ydst + col0, Ysrc + col0, Bsum + col0, M, Ksum, d, d_out, ws, ws};
      g.job[j++] = SplitJob{pinv + (int64_t)P * kBb * kBb, delta_w + (int64_t)P * kBb * d_out + col0, nullptr,
                            Bp + col0, Kp, Kp, kBb, d_out, ws, dws};
      g.n_jobs = j;
      g.N = ncols;
      g.layers = nl;
      g.ldb = d_out;
      g.lb = ws;
      return launch_split<true>(g, st);
    };
    hipError_t e;
    // the first step reads the right-hand side C itself (Y = C before any update)
    e = fwd_launch(up(0, 1), yblk(Y, 1), yblk(C, 1), d - kBb, C, kblk(0), 0, C, kblk(0));
    if (e != hipSuccess) return e;
    for (int I = 1; I < nb; I += 2) {
      if (I + 1 == nb) {
        e = fwd_launch(nullptr, Y, Y, 0, Y, 0, I, yblk(Y, I), kblk(I));
        if (e != hipSuccess) return e;
        break;
      }
      e = fwd_launch(up(I, I + 1), yblk(Y, I + 1), yblk(Y, I + 1), kblk(I + 1), yblk(Y, I), kBb, I, yblk(Y, I),
                     kBb);
      if (e != hipSuccess) return e;
      const int below = d - (I + 2) * kBb;
      e = fwd_launch(below > 0 ? up(I, I + 2) : nullptr, below > 0 ? yblk(Y, I + 2) : Y,
                     below > 0 ? yblk(Y, I + 2) : Y, max(below, 0), yblk(Y, I), kBb + kblk(I + 1), I + 1,
                     yblk(Y, I + 1), kblk(I + 1));
      if (e != hipSuccess) return e;
    }
    // backward sweep: dW_I -= Lh_JI^T dW_J (I < J), from the last block down in
    // pairs (J, J-1): one launch finishes dW_{J-1}, the next updates every earlier
    // block with both (rows (J-1)*256 .. of L, depth 512); rows from row0 on
    auto bwd_launch = [&](int J, int M, int K, int row0) -> hipError_t {
      SplitArgs g = {};
      float* dst = delta_w + (int64_t)row0 * d_out + col0;
      g.job[0] = SplitJob{L + (int64_t)row0 * d + (int64_t)J * kBb, dst, dst, yblk(delta_w, J) + col0, M, K, d, d_out, ws, dws};
      g.n_jobs = 1;
      g.N = ncols;
      g.layers = nl;
      g.ldb = d_out;
      g.lb = dws;
      return launch_split<false>(g, st);
    };
    for (int J = nb - 1; J >= 1; J -= 2) {
      e = bwd_launch(J, kBb, kblk(J), (J - 1) * kBb);
      if (e != hipSuccess) return e;
      if (J - 1 >= 1) {
        e = bwd_launch(J - 1, (J - 1) * kBb, kBb + kblk(J), 0);
        if (e != hipSuccess) return e;
      }
    }
    return hipSuccess;
  };
  {
    SideStream* side = d_out >= 2 * kSweepCols ? side_stream(d) : nullptr;
    hipError_t e;
    if (side != nullptr) {
      std::lock_guard<std::mutex> lock(g_side_mu);
      const int half = (d_out / 2 + kSweepCols - 1) / kSweepCols * kSweepCols;
      if ((e = hipEventRecord(side->fork, stream)) != hipSuccess) return e;
      if ((e = hipStreamWaitEvent(side->s, side->fork, 0)) != hipSuccess) return e;
      if ((e = sweeps(0, half, stream)) != hipSuccess) return e;
      if ((e = sweeps(half, d_out - half, side->s)) != hipSuccess) return e;
      if ((e = hipEventRecord(side->join, side->s)) != hipSuccess) return e;
      if ((e = hipStreamWaitEvent(stream, side->join, 0)) != hipSuccess) return e;
    } else if ((e = sweeps(0, d_out, stream)) != hipSuccess) {
      return e;
    }
  }
  // the P_I area is free once the forward sweep has run: it holds the partial sums
  const int64_t n = (int64_t)d * d_out;
  hipLaunchKernelGGL(eps_partial_kernel, dim3(kEpsBlocks, nl), dim3(kThreads), 0, stream, delta_w, C, n,
                     (double*)pinv, ws, dws);
  hipLaunchKernelGGL(eps_final_kernel, dim3(1, nl), dim3(kThreads), 0, stream, (const double*)pinv, kEpsBlocks,
                     w.scalars, (double)lambda, (const int*)w.status, w.eps_out, w.status_out, ws);
  return hipGetLastError();
}

}  // namespace ispa
