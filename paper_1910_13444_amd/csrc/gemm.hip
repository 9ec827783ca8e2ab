// Matrix-core (MFMA) kernels of the PI-GAN step for gfx950.
//
// k_gemm_nt  : C_k = X_k . W^T for the C jet streams of a tile of points,
//              with three fused epilogues:
//   EPI_FWD  hidden-layer forward: adds the bias to the value stream, applies
//            tanh and carries the spatial derivatives forward
//              h = t, h'_i = s a'_i, h''_i = s a''_i + s' (a'_i)^2
//            (chain rule of the generator's induced derivative network,
//            Sec. III.B.1); writes the pre-activations (kept for the reverse
//            pass) and the activations.
//   EPI_BWD  reverse pass: the product is dH of the layer below; the epilogue
//            turns it into that layer's pre-activation cotangents
//              g_a   = s g_h + sum_i s' a'_i g_h'_i + (s' a''_i + s'' a'_i^2) g_h''_i
//              g_a'_i = s g_h'_i + 2 s' a'_i g_h''_i,   g_a''_i = s g_h''_i
//   EPI_DF   reverse pass through the discriminator's first layer for the
//            fake snapshots: writes -dL_D/dF (the adversarial generator loss
//            is the negated critic term) into the generators' sensor-row
//            cotangents, or into a per-critic input-cotangent array.
//   Residual blocks of a shared trunk add the skip activations (forward) and
//   the skip cotangent (reverse) in the same epilogues.
// k_gemm_dw  : dW = sum_rows dA^T H (split over rows, fp32 partials), plus
//              the bias cotangent sum over the value rows.
// The split partials are summed in fp64, in a fixed order, by k_colsum.
//
// Tiles: a 64-lane wave owns 32 points x 32*NT columns for every stream; the
// block is WM x WN waves.  The MFMA computes W . X^T so that a lane holds one
// point and runs of four columns (vector stores, lane-local derivative
// carry).  Operands are staged through LDS in 64-byte k-slices (swizzled
// segments, conflict-free writes and fragment reads): 16-bit layers of 128
// columns and more load them straight into LDS, two slices (a whole 128-byte
// line of every row) per stage, the others prefetch the next slices into
// registers while the current one is multiplied.
#include "common.h"

namespace pigan {

// Operand stages of k_gemm_nt: 64-byte rows (one k-slice) with the four
// 16-byte segments of row r stored in the order s ^ ((r >> 2) & 3).  The
// fragment reads (32 consecutive rows, one segment) and the stage writes (four
// lanes per row) are then both free of bank conflicts (measured with the
// LDS bank-conflict counter; a padded pitch without the swizzle conflicted on
// the writes).
static constexpr int LDS_PITCH = 64;
// registers of accumulators, fragments and saved pre-activations up to which the
// ring kernels issue their fragment reads one chunk ahead (PIPE)
static constexpr int PIPE_REGS = 200;
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int lds_seg(int row, int seg) { return row * LDS_PITCH + ((seg ^ ((row >> 2) & 3)) << 4); }

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Map hardware block b to a logical tile so that every XCD walks one
// contiguous range of logical tiles: blocks that share an operand tile run on
// the same XCD at about the same time.  Bijective for any block count.
__device__ __forceinline__ int64_t xcd_remap(int64_t b, int64_t nb) {
  const int64_t q = nb / 8, r = nb % 8;
  const int64_t x = b % 8, local = b / 8;
  return x < r ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// four consecutive elements in the storage type (8 bytes in bf16/fp16, 16 in fp32)
template <class T>
__device__ __forceinline__ void store4(T* p, const float* v) {
  if (sizeof(T) == 2) {
    uint2 raw;
    T* e = (T*)&raw;
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = Elem<T>::from_f(v[i]);
    *(uint2*)p = raw;
  } else {
    *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
  }
}

template <class T>
__device__ __forceinline__ void load4(const T* p, float* v) {
  if (sizeof(T) == 2) {
    const uint2 raw = *(const uint2*)p;
    const T* e = (const T*)&raw;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = Elem<T>::to_f(e[i]);
  } else {
    const float4 a = *(const float4*)p;
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  }
}

// A 32 x 32 product fragment against rows in memory.  The matrix core leaves
// lane l with point l & 31 and four consecutive columns per register group q
// (8 q + 4 (l >> 5) ..).  Two lane exchanges turn that into 16-byte row pieces
// of which four lanes (l, l + 32, l + 16, l + 48) cover 64 consecutive bytes:
// v_permlane32_swap_b32 (16-bit storage only: gathers eight columns per lane),
// then v_permlane16_swap_b32, which trades the second piece of point p with
// the first piece of point p + 16.  Piece pair i, half j of a lane is then
// point (l & 15) + 16 j, columns FragPos::col(i) ...  Both swaps are their own
// inverse, so loads run the same steps backwards.  (32-byte pieces, without
// the second exchange, made the forward stores of five streams slower than
// staging whole rows through LDS: 1.82 against 1.76 ms at K = N = 512,
// 256,064 points; 64-byte pieces take neither barrier nor LDS.)
template <class T> struct FragRaw { u32x4 w[sizeof(T) == 2 ? 1 : 2][2]; };

__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap16(u32x4& a, u32x4& b) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const auto r = __builtin_amdgcn_permlane16_swap(a[e], b[e], false, false);
    a[e] = r[0];
    b[e] = r[1];
  }
}

// first column of the lane's piece in pair i (of a fragment's 32 columns)
template <class T>
__device__ __forceinline__ int frag_col(int lane, int i) {
  return sizeof(T) == 2 ? 16 * ((lane >> 4) & 1) + 8 * (lane >> 5) : 16 * i + 8 * ((lane >> 4) & 1) + 4 * (lane >> 5);
}

// both values rounded to the storage type, together: converted one at a time,
// fp16 results come from v_fma_mixlo_f16, which rounds the last operation to
// 16 bits at once and not after its fp32 rounding (80 of them in the five-stream
// reverse epilogue: other values in rare cases, and two instructions a pair)
template <class T>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef T T2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), T2));
}

// products layout -> pieces
template <class T>
__device__ __forceinline__ void frag_pack(FragRaw<T>& f, const f32x16& v) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int b = 8 * j;
      uint32_t a0 = pack2<T>(v[b], v[b + 1]), a1 = pack2<T>(v[b + 2], v[b + 3]);
      uint32_t b0 = pack2<T>(v[b + 4], v[b + 5]), b1 = pack2<T>(v[b + 6], v[b + 7]);
      swap32(a0, b0);
      swap32(a1, b1);
      f.w[0][j] = u32x4{a0, a1, b0, b1};
    }
    swap16(f.w[0][0], f.w[0][1]);
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) f.w[i][j][e] = __float_as_uint(v[8 * i + 4 * j + e]);
      swap16(f.w[i][0], f.w[i][1]);
    }
  }
}

// pieces -> products layout: first the lane exchanges of the whole fragment,
// then the lane's values of register group q
template <class T>
__device__ __forceinline__ void frag_unswap(FragRaw<T>& f) {
#pragma unroll
  for (int i = 0; i < (sizeof(T) == 2 ? 1 : 2); ++i) swap16(f.w[i][0], f.w[i][1]);
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        uint32_t x = f.w[0][j][c], y = f.w[0][j][2 + c];
        swap32(x, y);
        f.w[0][j][c] = x;
        f.w[0][j][2 + c] = y;
      }
  }
}
template <class T>
__device__ __forceinline__ void frag_group(const FragRaw<T>& f, int q, float* v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (sizeof(T) == 2)
      v[e] = Elem<T>::to_f(__builtin_bit_cast(T, (uint16_t)(f.w[0][q >> 1][2 * (q & 1) + (e >> 1)] >> (16 * (e & 1)))));
    else
      v[e] = __uint_as_float(f.w[q >> 1][q & 1][e]);
  }
}

// Barrier for data exchanged through LDS only.  __syncthreads() also fences
// global memory, which makes every wave wait for all of its outstanding global
// loads (s_waitcnt vmcnt(0)) and so defeats loads prefetched stages ahead;
// here only the LDS writes must be complete before the barrier.
__device__ __forceinline__ void lds_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Jet carries through tanh of one (point, column); index k runs over the
// streams: value, d/dx_1..d/dx_ND1, d^2/dx_1^2..d^2/dx_ND2^2.
// Forward: pre-activations in, activations out.
template <int ND1, int ND2, bool X64 = false>
__device__ __forceinline__ void jet_fwd(float* v) {
  float tt, s;
  tanh_pair<X64>(v[0], tt, s);
  const float sp = -2.0f * tt * s;
#pragma unroll
  for (int i = 0; i < ND2; ++i) v[1 + ND1 + i] = s * v[1 + ND1 + i] + sp * v[1 + i] * v[1 + i];
#pragma unroll
  for (int i = 0; i < ND1; ++i) v[1 + i] *= s;
  v[0] = tt;
}

// Reverse: activation cotangents in, pre-activation cotangents out, given the
// saved pre-activations ap.
template <int ND1, int ND2, bool X64 = false>
__device__ __forceinline__ void jet_bwd(float* g, const float* ap) {
  float tt, s;
  tanh_pair<X64>(ap[0], tt, s);
  const float sp = -2.0f * tt * s;
  const float spp = 2.0f * s * (3.0f * tt * tt - 1.0f);
  float ga = s * g[0];
#pragma unroll
  for (int i = 0; i < ND1; ++i) ga += sp * ap[1 + i] * g[1 + i];
#pragma unroll
  for (int i = 0; i < ND2; ++i) ga += (sp * ap[1 + ND1 + i] + spp * ap[1 + i] * ap[1 + i]) * g[1 + ND1 + i];
#pragma unroll
  for (int i = 0; i < ND1; ++i) {
    float v = s * g[1 + i];
    if (i < ND2) v += 2.0f * sp * ap[1 + i] * g[1 + ND1 + i];
    g[1 + i] = v;
  }
#pragma unroll
  for (int i = 0; i < ND2; ++i) g[1 + ND1 + i] *= s;
  g[0] = ga;
}

// Wait until at most N vector-memory operations of this wave are outstanding
// (N is an immediate).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// RING (16-bit types): the operand stages move from global memory straight
// into two LDS buffers (global_load_lds_dwordx4, no register staging), one
// stage ahead of the multiply.  A stage is 128 bytes of every row, loaded as
// two 64-byte slices back to back: a cache line then crosses from L2 once
// (measured with every block reading L2-resident rows: 18.3 TB/s over the chip
// for single 64-byte slices, 34.8 TB/s in pairs).
// OUT (with RING): the output layer fused in place of the activations' store
// (nt_ring_out_ok: where this pays, with figures).
// PM (fp32 storage only): products from bf16 pieces of the fp32 operands
// (ProdMode).
// p.kx > 0 (two-term weights): operand X is kx wide, the weight rows
// [W_hi | W_lo] are 2 kx wide and X is read twice: all high terms are added in
// the order of k, then all low ones.  (Staging a slice of X once for both terms
// saves its second read, but adds the low terms beside partial sums of the high
// ones: where those cancel, the low terms are rounded away.)
template <class T, int ND1, int ND2, int WM, int WN, int MT, int NT, int EPI, int OCC, bool DB = (OCC >= 2),
          bool RING = false, int PM = PM_NATIVE, int NB = 2, int SL = 1, bool OUT = false>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC)))
k_gemm_nt(const NtArgs<T> p) {
  constexpr int C = 1 + ND1 + ND2;
  constexpr int BM = 32 * MT * WM;
  constexpr int BN = 32 * NT * WN;
  constexpr int NTH = 64 * WM * WN;
  constexpr int ES = (int)sizeof(T);
  constexpr int KS = 64 / ES;                      // k values per stage
  constexpr int NCH = 64 / (16 * ES);              // 16-wide chunks per stage
  constexpr int ROWS = C * BM + BN;
  constexpr int SLICE = ROWS * LDS_PITCH;          // bytes of one 64-byte k slice of the operands
  constexpr int STAGE = SL * SLICE;                // register-staged: SL slices per stage
  constexpr int PIECES = ROWS * 4 * SL;
  constexpr int PPT = (PIECES + NTH - 1) / NTH;
  constexpr int XBUF = 2 * C * BM * LDS_PITCH, WBUF = 2 * BN * LDS_PITCH;   // RING buffers
  constexpr int OUTB = PM == PM_F64 ? BM * 65 * 4 : 0;   // fp64 products are re-laid out through LDS
  constexpr int LDSB = RING ? 2 * (XBUF + WBUF) : (2 * STAGE > OUTB ? 2 * STAGE : OUTB);
  static_assert(!RING || (ES == 2 && PM == PM_NATIVE), "direct-to-LDS stages: 16-bit types");
  static_assert(PM == PM_NATIVE || ES == 4, "split products: fp32 storage");
  static_assert(!OUT || (RING && EPI == EPI_FWD), "fused output layer: ring kernels, forward products");
  // fp32 mode (fp32 storage, products not split into bf16): tanh in fp64
  constexpr bool X64 = ES == 4 && PM != PM_SPLIT2;
  typedef typename Elem<T>::frag frag;
  __shared__ __attribute__((aligned(16))) char lds[LDSB];

  const int g = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % WM;
  const int wn = wave / WM;
  // logical tile: column tiles fastest, so the blocks reading one tile of
  // activations run together on one XCD and share it through its L2
  const int ntn = (p.N + BN - 1) / BN;
  const int64_t lt = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t m0 = (lt / ntn) * BM;
  const int n0 = (int)(lt % ntn) * BN;
  const int64_t npts = p.seg.n_points;

  const char* Xb = (const char*)(p.X + g * p.x_g);
  const char* Wb = (const char*)(p.Wm + g * p.w_g);

  // each thread moves PPT 16-byte pieces of every stage: operand row piece>>2,
  // 16-byte segment piece&3 of its 64-byte k-slice.  The register ring
  // (NB > 2) loads unconditionally, so that the compiler can count the loads
  // in flight and wait only for the stage it stores (a load under a condition
  // makes it wait for all of them): points past the segment end and columns
  // past N read a clamped (valid) row, whose products are never stored, and
  // threads without a piece re-read the operand's first segment and drop it.
  // (Elsewhere the loads stay conditional: unconditional ones there moved the
  // staging registers of many kernels to scratch memory.)
  constexpr bool UNCOND = DB && NB > 2;
  const char* src[PPT];
  bool valid[PPT], isx[PPT];
#pragma unroll
  for (int i = 0; i < (RING ? 0 : PPT); ++i) {
    const int piece = tid + i * NTH;
    const int row = piece / (4 * SL), sg = piece % (4 * SL);
    valid[i] = UNCOND;
    isx[i] = row < C * BM || piece >= PIECES;   // a dropped re-read stays inside X's first row
    src[i] = Xb;
    if (piece < PIECES) {
      if (row < C * BM) {
        const int k = row / BM, pp = row % BM;
        int64_t pt = m0 + pp;
        valid[i] = UNCOND || pt < npts;
        if (UNCOND && pt > npts - 1) pt = npts - 1;
        src[i] = Xb + (p.seg.row0 + k * p.seg.plane + pt) * p.ldx * (int64_t)ES + sg * 16;
      } else {
        int n = n0 + row - C * BM;
        valid[i] = UNCOND || n < p.N;
        if (UNCOND && n > p.N - 1) n = p.N - 1;
        src[i] = Wb + (int64_t)n * p.ldw * (int64_t)ES + sg * 16;
      }
    }
  }

  // the lane's part of the outputs: hh selects the column half of every
  // fragment, mloc the point within the block (the epilogue's layout)
  const int hh = lane >> 5;
  auto mloc = [&](int u) { return 32 * (MT * wm + u) + (lane & 31); };
  auto ncol = [&](int t, int q) { return 32 * (wn * NT + t) + 8 * q + 4 * hh; };   // column within the block
  auto fcol = [&](int t) { return n0 + 32 * (wn * NT + t); };                      // first column of a fragment
  // point of the lane's half j of fragment u (frag_pack's layout)
  auto fpt = [&](int u, int j) { return m0 + 32 * (MT * wm + u) + (lane & 15) + 16 * j; };
  // the pieces of fragment (u, t) of stream k of an array laid out as the
  // outputs; points past the segment end and columns past N take valid elements
  // (one_row: the stream's single row, a_seeds)
  auto load_frag = [&](FragRaw<T>& f, const T* base, int u, int k, int t, bool one_row = false) {
    const int nb = fcol(t) < p.N ? fcol(t) : 0;
    const int64_t row0 = p.seg.row0 + (one_row ? p.seg.plane + k - 1 : k * p.seg.plane);
    const int64_t pmask = one_row ? 0 : -1;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int64_t pt = fpt(u, j);
      if (pt > npts - 1) pt = npts - 1;
      const T* row = base + g * p.o_g + (row0 + (pt & pmask)) * p.ldo + nb;
#pragma unroll
      for (int i = 0; i < (ES == 2 ? 1 : 2); ++i) f.w[i][j] = *(const u32x4*)(row + frag_col<T>(lane, i));
    }
  };

  // reverse pass: the saved pre-activations the epilogue needs.  PRE: where
  // the registers allow it they are read before the products, so that their
  // latency is covered by them
  constexpr bool PRE = EPI == EPI_BWD && RING && MT * C * NT * 24 <= 160;
  FragRaw<T> apre[PRE ? MT : 1][PRE ? C : 1][PRE ? NT : 1];
  if constexpr (PRE) {
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int k = 0; k < C; ++k) load_frag(apre[u][k][t], p.aprev, u, k, t, k > 0 && p.a_seeds);
    __builtin_amdgcn_sched_barrier(0);
  }

  f32x16 acc[MT][C][NT];
#pragma unroll
  for (int u = 0; u < MT; ++u)
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][k][t][r] = 0.0f;

  // stage kt of the weights is stage kxs(kt) of operand X (two-term weights
  // read X twice)
  const int nk = p.K / (KS * SL);
  const int nkx = p.kx > 0 ? p.kx / (KS * SL) : nk;
  auto kxs = [&](int kt) { return kt >= nkx ? kt - nkx : kt; };
  auto gload = [&](uint4* buf, int kt) {
    const int ktx = kxs(kt);
#pragma unroll
    for (int i = 0; i < PPT; ++i)
      buf[i] = (UNCOND || valid[i]) ? *(const uint4*)(src[i] + (int64_t)(isx[i] ? ktx : kt) * (64 * SL))
                                    : make_uint4(0u, 0u, 0u, 0u);
  };
  // PM_SPLIT2: each fp32 value of operand X is cut into its two bf16 pieces
  // once, as the stage is stored: a 64-byte stage row (16 k) then holds the
  // high pieces in segments 0-1 and the low pieces in segments 2-3, i.e. the
  // layout of a 16-bit stage whose first 16-wide chunk is the high part and
  // second the low part.  The weight rows arrive in that layout already (the
  // weight copies are split once per step), and are stored as loaded.
  auto lstore = [&](const uint4* buf, int stage) {
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int piece = tid + i * NTH;
      if (PIECES % NTH != 0 && piece >= PIECES) continue;
      const int row = piece / (4 * SL), sg = piece & 3;
      char* base = lds + stage * STAGE + (piece / 4 % SL) * SLICE;
      if (PM == PM_SPLIT2 && row < C * BM) {
        const float* v = (const float*)&buf[i];
        bf16 hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          hi[e] = (bf16)v[e];
          lo[e] = (bf16)(v[e] - (float)hi[e]);
        }
        *(uint2*)(base + lds_seg(row, sg >> 1) + (sg & 1) * 8) = __builtin_bit_cast(uint2, hi);
        *(uint2*)(base + lds_seg(row, 2 + (sg >> 1)) + (sg & 1) * 8) = __builtin_bit_cast(uint2, lo);
      } else {
        *(uint4*)(base + lds_seg(row, sg)) = buf[i];
      }
    }
  };
  // a fragment: 8 consecutive k of one row (16 bytes in 16-bit types, two
  // segments in fp32); every fragment row base is a multiple of 32, so the
  // segment swizzle of the lane's row is (lane >> 2) & 3
  const int gsw = (lane >> 2) & 3;
  auto frag_at = [&](const char* base, int row, int c) {
    if constexpr (ES == 2) {
      const int seg = 2 * c + (lane >> 5);
      return *(const frag*)(base + row * LDS_PITCH + ((seg ^ gsw) << 4));
    } else {
      const int seg = 2 * (lane >> 5);
      const u32x4 lo = *(const u32x4*)(base + row * LDS_PITCH + ((seg ^ gsw) << 4));
      const u32x4 hi = *(const u32x4*)(base + row * LDS_PITCH + (((seg + 1) ^ gsw) << 4));
      const u32x8 w = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      return __builtin_bit_cast(frag, w);
    }
  };
  // the high (c = 0) or low (c = 1) bf16 pieces of a PM_SPLIT2 fragment
  auto piece_at = [&](const char* base, int row, int c) {
    return *(const bf16x8*)(base + row * LDS_PITCH + (((2 * c + (lane >> 5)) ^ gsw) << 4));
  };
  auto compute_slice = [&](const char* base) {
    if constexpr (PM == PM_SPLIT2) {
      bf16x8 bp[NT][2];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) bp[t][c] = piece_at(base, C * BM + 32 * (wn * NT + t) + (lane & 31), c);
#pragma unroll
      for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) {
          bf16x8 ap[2];
#pragma unroll
          for (int c = 0; c < 2; ++c) ap[c] = piece_at(base, k * BM + 32 * (MT * wm + u) + (lane & 31), c);
#pragma unroll
          for (int t = 0; t < NT; ++t) mma_split(acc[u][k][t], bp[t], ap);
        }
      return;
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      frag bfr[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) bfr[t] = frag_at(base, C * BM + 32 * (wn * NT + t) + (lane & 31), c);
#pragma unroll
      for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) {
          const frag afr = frag_at(base, k * BM + 32 * (MT * wm + u) + (lane & 31), c);
#pragma unroll
          for (int t = 0; t < NT; ++t) Elem<T>::mma(acc[u][k][t], bfr[t], afr);   // rows: columns n; cols: points
        }
    }
  };
  auto compute = [&](int stage) {
#pragma unroll
    for (int i = 0; i < SL; ++i) compute_slice(lds + stage * STAGE + i * SLICE);
  };
  static_assert(SL == 1 || PM == PM_SPLIT2, "wider stages: split products");
  // PM_F64 (one fragment per wave and stream: 32 points x 32 columns, 2 x 2
  // blocks of the 16 x 16 fp64 product, whose lane l holds rows
  // (l >> 4) + 4 r and column l & 15 of a block)
  static_assert(PM != PM_F64 || (MT == 1 && NT == 1 && C <= 2), "fp64 products: one fragment per wave");
  f64x4 accd[PM == PM_F64 ? C : 1][2][2];
  if constexpr (PM == PM_F64) {
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) accd[k][a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  }
  // fp32 element kx (0..15) of LDS stage row r
  auto lds_f = [&](const char* base, int r, int kx) {
    return (double)*(const float*)(base + lds_seg(r, kx >> 2) + (kx & 3) * 4);
  };
  auto compute64 = [&](int stage) {
    const char* base = lds + stage * STAGE;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int kx = 4 * kk + (lane >> 4);
      double wv[2];
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) wv[nb] = lds_f(base, C * BM + 32 * wn + 16 * nb + (lane & 15), kx);
#pragma unroll
      for (int k = 0; k < C; ++k)
#pragma unroll
        for (int pb = 0; pb < 2; ++pb) {
          const double xv = lds_f(base, k * BM + 32 * wm + 16 * pb + (lane & 15), kx);
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            accd[k][nb][pb] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[nb], xv, accd[k][nb][pb], 0, 0, 0);
        }
    }
  };
  if constexpr (RING) {
    // One DMA instruction of a wave fills 1 KB of LDS, lane l at byte 16 l:
    // 16 rows of a slice (row 16 g + l / 4, physical segment l % 4, holding
    // the logical segment (l % 4) ^ ((row >> 2) & 3) of the swizzled layout).
    // The row groups of X and of the weights are dealt to the waves
    // round-robin.  A group lies in one stream of X, or in the weights: its
    // address is a wave-uniform base plus a 32-bit lane offset.  Points past
    // the segment end and columns past N read a clamped (valid) row: their
    // products are never stored.
    constexpr int NW = NTH / 64;
    constexpr int XG = C * BM / 16, WG = BN / 16;
    constexpr int XPW = (XG + NW - 1) / NW, WPW = (WG + NW - 1) / NW;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sgl = ((lane & 3) ^ ((lane >> 4) & 3)) * 16;   // the lane's logical segment (row >> 2 = lane >> 4 mod 4)
    const char* xsrc[XPW];
    uint32_t xoff[XPW];
    const char* wsrc[WPW];
    uint32_t woff[WPW];
#pragma unroll
    for (int i = 0; i < XPW; ++i) {
      const int row0 = (wv + i * NW) * 16;
      const int k = row0 / BM;
      int64_t pp = row0 % BM + (lane >> 2);
      if (pp > npts - 1 - m0) pp = npts - 1 - m0;
      xsrc[i] = Xb + (p.seg.row0 + k * p.seg.plane + m0) * p.ldx * (int64_t)ES;
      xoff[i] = (uint32_t)(pp * p.ldx * ES) + sgl;
    }
#pragma unroll
    for (int i = 0; i < WPW; ++i) {
      int n = (wv + i * NW) * 16 + (lane >> 2);
      if (n > p.N - 1 - n0) n = p.N - 1 - n0;
      wsrc[i] = Wb + (int64_t)n0 * p.ldw * (int64_t)ES;
      woff[i] = (uint32_t)(n * p.ldw * ES) + sgl;
    }
    char* const xlds = lds;
    char* const wlds = lds + 2 * XBUF;
    const int ns = p.K / 64;
    const int nx = p.kx > 0 ? p.kx / 64 : ns;
    auto issue = [&](int s) {
      const int sx = s >= nx ? s - nx : s;
#pragma unroll
      for (int i = 0; i < WPW; ++i) {
        if (WG % NW != 0 && wv + i * NW >= WG) break;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          __builtin_amdgcn_global_load_lds((const void*)(wsrc[i] + (int64_t)s * 128 + 64 * h + woff[i]),
                                           (lds_ptr_t)(wlds + (s & 1) * WBUF + h * (WBUF / 2) + (wv + i * NW) * 1024),
                                           16, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < XPW; ++i) {
        if (XG % NW != 0 && wv + i * NW >= XG) break;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          __builtin_amdgcn_global_load_lds((const void*)(xsrc[i] + (int64_t)sx * 128 + 64 * h + xoff[i]),
                                           (lds_ptr_t)(xlds + (s & 1) * XBUF + h * (XBUF / 2) + (wv + i * NW) * 1024),
                                           16, 0, 0);
      }
    };
    frag xf[2][MT][C], wf[2][NT];
    auto read_chunk = [&](int s, int c, int b) {
      const char* xb = xlds + (s & 1) * XBUF + (c >> 1) * (XBUF / 2);
      const char* wb = wlds + (s & 1) * WBUF + (c >> 1) * (WBUF / 2);
#pragma unroll
      for (int t = 0; t < NT; ++t) wf[b][t] = frag_at(wb, 32 * (wn * NT + t) + (lane & 31), c & 1);
#pragma unroll
      for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k) xf[b][u][k] = frag_at(xb, k * BM + 32 * (MT * wm + u) + (lane & 31), c & 1);
    };
    auto products = [&](int b) {
#pragma unroll
      for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k)
#pragma unroll
          for (int t = 0; t < NT; ++t) Elem<T>::mma(acc[u][k][t], wf[b][t], xf[b][u][k]);   // rows: columns n; cols: points
    };
    // PIPE (where the registers allow it): the reads of a 16-wide chunk's
    // fragments are issued before the products of the chunk before, across the
    // stage barrier too.  They do not stay ahead: while a direct-to-LDS load is
    // outstanding the compiler drains every LDS read before a use (all 212
    // waits of these kernels' product loops are lgkmcnt(0)), so two of a stage's
    // four chunks wait for their successor's fragments as well, and what is
    // gained is one wait for two chunks.  Without it: seven streams at 128
    // columns 1.40 -> 1.46 ms (3-D residual), widths 256 to 1024 within 1 %.
    constexpr bool PIPE = MT * C * NT * 16 + 8 * (MT * C + NT) + (PRE ? 8 * MT * C * NT : 0) <= PIPE_REGS;
    if constexpr (PIPE) {
      issue(0);
      wait_vmcnt<0>();
      lds_sync();
      if (ns > 1) issue(1);
      read_chunk(0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      for (int s = 0; s < ns; ++s) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          read_chunk(s, c + 1, (c + 1) & 1);
          __builtin_amdgcn_sched_barrier(0);
          products(c & 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (s + 1 < ns) {
          wait_vmcnt<0>();
          lds_sync();   // stage s + 1 has landed for every wave, stage s has been read by every wave
          if (s + 2 < ns) issue(s + 2);
          read_chunk(s + 1, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        products(1);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      issue(0);
      for (int s = 0; s < ns; ++s) {
        wait_vmcnt<0>();
        lds_sync();   // stage s has landed for every wave, and every wave is done with stage s - 1
        if (s + 1 < ns) issue(s + 1);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          read_chunk(s, c, 0);
          products(0);
        }
      }
    }
  } else if constexpr (DB && NB > 2) {
    // two LDS stages and a ring of NB register buffers: buffer b holds the
    // stages kt = b (mod NB), so the global loads of stage kt + NB are issued
    // while stage kt is multiplied.  Loads are unconditional (stage index
    // clamped), so the compiler's waits are static counts.
    uint4 bufs[NB][PPT];
    const int last = nk - 1;
#pragma unroll
    for (int b = 0; b < NB; ++b) gload(bufs[b], b < last ? b : last);
    lstore(bufs[0], 0);
    gload(bufs[0], NB < last ? NB : last);
    lds_sync();
    // UR rounds of the ring per loop pass: the compiler drains every load in
    // flight once per pass (its wait analysis does not carry the ring across
    // the back edge), so longer passes drain less often
    constexpr int UR = 4;
    for (int k0 = 0; k0 < nk; k0 += NB * UR) {
#pragma unroll
      for (int u = 0; u < NB * UR; ++u) {
        const int kt = k0 + u;
        if (kt >= nk) break;
        if constexpr (PM == PM_F64) compute64(kt & 1); else compute(kt & 1);
        __builtin_amdgcn_sched_barrier(0);
        if (kt + 1 < nk) lstore(bufs[(u + 1) % NB], (kt + 1) & 1);
        gload(bufs[(u + 1) % NB], kt + 1 + NB < last ? kt + 1 + NB : last);
        lds_sync();
      }
    }
  } else if constexpr (DB) {
    // two LDS stages, two register buffers: the global loads of stage kt+2
    // are issued before stage kt is multiplied; one barrier per stage
    // prefetches are unconditional (the stage index is clamped; loads past
    // the last stage are never stored): conditional loads would force
    // register copies that wait for the data
    uint4 b0[PPT], b1[PPT];
    gload(b0, 0);
    lstore(b0, 0);
    gload(b1, nk > 1 ? 1 : 0);
    lds_sync();
    for (int kt = 0; kt < nk; kt += 2) {
      gload(b0, kt + 2 < nk ? kt + 2 : nk - 1);
      if constexpr (PM == PM_F64) compute64(0); else compute(0);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 1 < nk) lstore(b1, 1);
      lds_sync();
      if (kt + 1 >= nk) break;
      gload(b1, kt + 3 < nk ? kt + 3 : nk - 1);
      if constexpr (PM == PM_F64) compute64(1); else compute(1);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 2 < nk) lstore(b0, 0);
      lds_sync();
    }
  } else {
    // large tiles (one wave per SIMD): two LDS stages, one register buffer
    // loaded one stage ahead
    uint4 b0[PPT];
    gload(b0, 0);
    lstore(b0, 0);
    lds_sync();
    for (int kt = 0; kt < nk; ++kt) {
      gload(b0, kt + 1 < nk ? kt + 1 : nk - 1);
      if constexpr (PM == PM_F64) compute64(kt & 1); else compute(kt & 1);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 1 < nk) lstore(b0, (kt + 1) & 1);
      lds_sync();
    }
  }
  if constexpr (PM == PM_F64) {
    // each stream through LDS, [point][column] floats (pitch 65), into the
    // lane layout of the fp32 fragments the epilogue reads
    float* tl = (float*)lds;
    lds_sync();
#pragma unroll
    for (int k = 0; k < C; ++k) {
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int pb = 0; pb < 2; ++pb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            tl[(32 * wm + 16 * pb + (lane & 15)) * 65 + 32 * wn + 16 * nb + (lane >> 4) + 4 * r] =
                (float)accd[k][nb][pb][r];
      lds_sync();
#pragma unroll
      for (int r = 0; r < 16; ++r)
        acc[0][k][0][r] = tl[(32 * wm + (lane & 31)) * 65 + 32 * wn + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)];
      lds_sync();
    }
  }

  // ---- epilogue.  The products were formed as W . X^T, so lane (lane & 31)
  // owns one point of each of its MT point sub-tiles and, in register group q
  // (regs 4q..4q+3), four consecutive columns 8q + 4*(lane >> 5) + 0..3 of
  // every 32x32 tile: all jet streams of a (point, column) sit in the same
  // lane.  Results leave straight from the registers as 16-byte row pieces
  // (store_rows): staging every stream through LDS took two barriers per
  // stream and array, which on the one-block-per-CU tiles nothing overlapped.
  if (EPI == EPI_DF) {
    const int64_t ldY = p.sY_ld > 0 ? p.sY_ld : p.nY, ldU = p.sU_ld > 0 ? p.sU_ld : p.nU;
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      const int64_t pt = m0 + mloc(u);
      if (pt >= npts) continue;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int n = n0 + ncol(t, q) + e;
            const float v = p.df_sign * acc[u][0][t][4 * q + e];
            if (n < p.nY) p.seedY[g * p.sY_g + pt * ldY + n] = v;
            else if (n < p.nY + p.nU) p.seedU[g * p.sU_g + pt * ldU + p.sU_off + (n - p.nY)] = v;
          }
    }
    return;
  }

  // writes / adds a [points x columns] array of every stream, laid out as the
  // outputs (N is a multiple of 32 here: a fragment's columns are all valid or
  // none)
  auto store_rows = [&](T* dst, int u, int t) {
    if (fcol(t) >= p.N) return;
    const int64_t p0 = fpt(u, 0), p1 = fpt(u, 1);
#pragma unroll
    for (int k = 0; k < C; ++k) {
      FragRaw<T> f;
      frag_pack<T>(f, acc[u][k][t]);
      T* row = dst + g * p.o_g + (p.seg.row0 + k * p.seg.plane + p0) * p.ldo + fcol(t);
#pragma unroll
      for (int i = 0; i < (ES == 2 ? 1 : 2); ++i) {
        if (p0 < npts) *(u32x4*)(row + frag_col<T>(lane, i)) = f.w[i][0];
        if (p1 < npts) *(u32x4*)(row + 16 * p.ldo + frag_col<T>(lane, i)) = f.w[i][1];
      }
    }
  };
  auto load_rows = [&](FragRaw<T>* raw, const T* src, int u, int t, bool seeds = false) {
#pragma unroll
    for (int k = 0; k < C; ++k) load_frag(raw[k], src, u, k, t, k > 0 && seeds);
    __builtin_amdgcn_sched_barrier(0);   // all in flight together
  };
  auto add_row = [&](FragRaw<T>& raw, int u, int k, int t) {
    frag_unswap<T>(raw);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[4];
      frag_group<T>(raw, q, v);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[u][k][t][4 * q + e] += v[e];
    }
  };
  auto add_rows = [&](FragRaw<T>* raw, int u, int t) {
#pragma unroll
    for (int k = 0; k < C; ++k) add_row(raw[k], u, k, t);
  };

  if (EPI == EPI_FWD) {
    // pre-activations (bias on the value stream), then activations in place:
    //   h = t, h'_i = s a'_i, h''_i = s a''_i + s' (a'_i)^2
    // (all biases of a lane are read together: behind a check of its own, each
    // of the up to 32 loads was waited for by itself, about a third of a
    // block's time at K = 512)
    // fused output layer: w_out . h over the lane's columns, the activations
    // as stored
    float ys[OUT ? MT : 1][OUT ? C : 1][OUT ? NT : 1];
    constexpr int HPITCH = 128 * ES + 16;          // of an LDS row of 128 activations
    static_assert(!OUT || (BN == 128 && BM == 32 && NTH == 256 && C * BM * HPITCH <= LDSB), "fused output layer: 128 columns per block");
    if (OUT) lds_sync();                           // the stages have been read
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float bv[16];
      {
        // columns past N take the first biases (their results are never stored)
        const float* bp = p.bias + g * p.b_g + (fcol(t) < p.N ? fcol(t) : 0) + 4 * hh;
#pragma unroll
        for (int r = 0; r < 16; ++r) bv[r] = bp[8 * (r >> 2) + (r & 3)];
      }
#pragma unroll
      for (int u = 0; u < MT; ++u) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][0][t][r] += bv[r];
        // (the residual rows are read ahead of the tanh where they fit)
        constexpr bool AHEAD = MT * C * NT * 16 < 160;
        FragRaw<T> sk[AHEAD ? C : 1];
        if constexpr (AHEAD && !OUT) {
          if (p.skip) load_rows(sk, p.skip, u, t);
        }
        if (p.out_a) store_rows(p.out_a, u, t);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float v[C];
#pragma unroll
          for (int k = 0; k < C; ++k) v[k] = acc[u][k][t][r];
          jet_fwd<ND1, ND2, X64>(v);
#pragma unroll
          for (int k = 0; k < C; ++k) acc[u][k][t][r] = v[k];
          if (MT * C * NT * 16 >= 160 && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (OUT && p.N == 128) {
          // whole rows in the block: the activations as stored, into LDS
#pragma unroll
          for (int k = 0; k < C; ++k) {
            FragRaw<T> f;
            frag_pack<T>(f, acc[u][k][t]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
              *(u32x4*)(lds + (k * BM + 32 * (MT * wm + u) + (lane & 15) + 16 * j) * HPITCH +
                        (32 * (wn * NT + t) + frag_col<T>(lane, 0)) * ES) = f.w[0][j];
          }
        } else if constexpr (OUT) {
          // (N is a multiple of 128: whole fragments)
          const float* wp = p.wout + g * p.wo_g + (fcol(t) < p.N ? fcol(t) : 0) + 4 * hh;
          float wo[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) wo[r] = wp[8 * (r >> 2) + (r & 3)];
#pragma unroll
          for (int k = 0; k < C; ++k) {
            float v = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) v += wo[r] * Elem<T>::to_f(Elem<T>::from_f(acc[u][k][t][r]));
            ys[u][k][t] = v;
          }
        } else {
          // residual block output: h_l = tanh carry + h_{l-2}, stream by stream
          if (p.skip) {
            if constexpr (AHEAD) {
              add_rows(sk, u, t);
            } else {
              // (a stream at a time: all five beside the accumulators spilled ten registers of the
              // 64 x 256 tile, also where there is no skip)
#pragma unroll
              for (int k = 0; k < C; ++k) {
                FragRaw<T> late;
                load_frag(late, p.skip, u, k, t);
                add_row(late, u, k, t);
                __builtin_amdgcn_sched_barrier(0);
              }
            }
          }
          store_rows(p.out_h, u, t);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (OUT) {
      if (p.N == 128) {
        // as k_out_fwd sums a row: the same bits
        lds_sync();
        const float* w = p.wout + g * p.wo_g;
        const int64_t pt = m0 + (tid >> 3);
        float v[C];
#pragma unroll
        for (int k = 0; k < C; ++k)
          v[k] = out_row_sum<T>((const T*)(lds + (k * BM + (tid >> 3)) * HPITCH), w, 128, tid & 7);
        if ((tid & 7) == 0 && pt < npts) {
#pragma unroll
          for (int k = 0; k < C; ++k)
            p.y[g * p.y_g + p.seg.row0 + k * p.seg.plane + pt] = v[k] + (k == 0 ? w[128] : 0.0f);
        }
        return;
      }
      // the lane halves, then the four fragments of each 128 columns in column
      // order, whatever waves and tiles hold them: the result does not depend
      // on the tile shape.  k_out_sum adds the groups of 128.
      float* red = (float*)lds;                    // [BN / 32][C][BM]
#pragma unroll
      for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int k = 0; k < C; ++k)
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float v = ys[u][k][t] + __shfl_xor(ys[u][k][t], 32);
            if (hh == 0) red[((wn * NT + t) * C + k) * BM + mloc(u)] = v;
          }
      lds_sync();
      for (int i = tid; i < (BN / 128) * C * BM; i += NTH) {
        const int gr = i / (C * BM), k = i / BM % C;
        const int64_t pt = m0 + i % BM;
        const float* f = red + (int64_t)gr * 4 * C * BM + i % (C * BM);
        const float v = ((f[0] + f[C * BM]) + f[2 * C * BM]) + f[3 * C * BM];
        if (pt >= npts || n0 + 128 * gr >= p.N) continue;
        p.ypart[g * p.yp_g + (int64_t)(n0 / 128 + gr) * C * npts + k * npts + pt] = v;
      }
    }
    return;
  }

  // reverse pass: the skip cotangent of a residual block's input, the total
  // kept for the skip below it, then the reverse carry in place: acc[k]
  // becomes the cotangent of the saved pre-activation a_k of the layer below
#pragma unroll
  for (int u = 0; u < MT; ++u) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (p.skip_g) {
        FragRaw<T> sk[C];
        load_rows(sk, p.skip_g, u, t);
        add_rows(sk, u, t);
      }
      FragRaw<T> raw[PRE ? 1 : C];
      if constexpr (!PRE) load_rows(raw, p.aprev, u, t, p.a_seeds);
      if (p.out_gh) store_rows(p.out_gh, u, t);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        if constexpr (PRE) frag_unswap<T>(apre[u][k][t]);
        else frag_unswap<T>(raw[k]);
      }
      // a register group at a time (all of a fragment would spill beside the
      // accumulators of the larger tiles)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float ap[C][4];
#pragma unroll
        for (int k = 0; k < C; ++k) {
          if constexpr (PRE) frag_group<T>(apre[u][k][t], q, ap[k]);
          else frag_group<T>(raw[k], q, ap[k]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float gv[C], av[C];
#pragma unroll
          for (int k = 0; k < C; ++k) {
            gv[k] = acc[u][k][t][4 * q + e];
            av[k] = ap[k][e];
          }
          jet_bwd<ND1, ND2, X64>(gv, av);
          // (fp64: an element's results are formed before the next one's; left
          // to itself the compiler evaluates one exponential of all sixteen
          // first and spills what is left of them, 8 and 25 registers with two
          // and four streams)
          if constexpr (X64) {
#pragma unroll
            for (int k = 0; k < C; ++k) asm volatile("" : "+v"(gv[k]));
          }
#pragma unroll
          for (int k = 0; k < C; ++k) acc[u][k][t][4 * q + e] = gv[k];
          if (X64 && e % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
        if (X64 || MT * C * NT * 16 >= 112 || q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
      store_rows(p.out_da, u, t);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// fused output layer over several groups of 128 columns: y = the groups' sums
// in order (+ b_out on the value stream)
__global__ void __launch_bounds__(256)
k_out_sum(const float* __restrict__ part, int64_t part_g, int groups, int64_t npts, int C, Seg seg,
          const float* __restrict__ wout, int64_t wo_g, int N, float* __restrict__ y, int64_t y_g) {
  const int g = blockIdx.z;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= C * npts) return;
  const float* p = part + g * part_g + i;
  float v = p[0];
  for (int t = 1; t < groups; ++t) v += p[(int64_t)t * C * npts];
  const int64_t k = i / npts;
  if (k == 0) v += wout[g * wo_g + N];
  y[g * y_g + seg.row0 + k * seg.plane + (i - k * npts)] = v;
}

// ---------------------------------------------------------------------------
// k_gemm_short: the fp64 products and epilogues of k_gemm_nt (fp32 storage)
// where a launch has few output tiles: a critic's batch, small sensor sets.
// There the tiled kernel is a serial chain of K stages on a few blocks (512
// rows, N = 256, K = 416: 32 blocks, 26 stages, 26.6 us; here 10.6).  A block owns 32 points x 32 columns and its NW waves share the
// contraction: each reads the operand fragments of its 16-wide chunks straight
// from global memory into registers, two chunks ahead, and the fp64 partial
// sums meet in LDS (added in wave order, rounded once).  The epilogue runs on
// 256 threads, four consecutive columns of one point each.
// ---------------------------------------------------------------------------
template <int ND1, int EPI, int NW>
__global__ void __launch_bounds__(64 * NW) k_gemm_short(const NtArgs<float> p) {
  constexpr int C = 1 + ND1;
  constexpr int SU = 2;                            // chunks in flight besides the ones being multiplied
  constexpr int PITCH = 34;                        // of one point's 32 columns
  __shared__ __attribute__((aligned(16))) double part[NW][32 * PITCH];
  const int g = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntn = p.N / 32;
  const int64_t lt = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t m0 = (lt / ntn) * 32;
  const int n0 = (int)(lt % ntn) * 32;
  const int64_t npts = p.seg.n_points;
  const int nch = p.K / 16;
  const int c0 = (int)((int64_t)nch * wave / NW), c1 = (int)((int64_t)nch * (wave + 1) / NW);

  // points past the end read the last one (their results are never stored)
  auto xrow = [&](int r, int k) {
    int64_t pt = m0 + r;
    if (pt > npts - 1) pt = npts - 1;
    return p.X + g * p.x_g + (p.seg.row0 + k * p.seg.plane + pt) * p.ldx;
  };
  f64x4 accd[C][2][2];
#pragma unroll
  for (int k = 0; k < C; ++k)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) accd[k][a][b] = f64x4{0.0, 0.0, 0.0, 0.0};

  {
    // lane: row l & 15 of each 16-row half, four k values 4 (l >> 4) of a
    // chunk; step j multiplies element j of every lane (both operands in the
    // same k order)
    const float* wr[2];
    const float* xr[C][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      wr[h] = p.Wm + g * p.w_g + (int64_t)(n0 + 16 * h + (lane & 15)) * p.ldw + 4 * (lane >> 4);
#pragma unroll
      for (int k = 0; k < C; ++k) xr[k][h] = xrow(16 * h + (lane & 15), k) + 4 * (lane >> 4);
    }
    f32x4 wb[2][SU][2], xb[2][SU][C][2];
    auto load = [&](int b, int c) {
#pragma unroll
      for (int i = 0; i < SU; ++i) {
        const int cc = c + i < c1 ? c + i : c1 - 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          wb[b][i][h] = *(const f32x4*)(wr[h] + cc * 16);
#pragma unroll
          for (int k = 0; k < C; ++k) xb[b][i][k][h] = *(const f32x4*)(xr[k][h] + cc * 16);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](int b, int c) {
#pragma unroll
      for (int i = 0; i < SU; ++i) {
        if (c + i >= c1) break;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int k = 0; k < C; ++k)
#pragma unroll
            for (int pb = 0; pb < 2; ++pb)
#pragma unroll
              for (int nb = 0; nb < 2; ++nb)
                accd[k][nb][pb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)wb[b][i][nb][j], (double)xb[b][i][k][pb][j],
                                                                       accd[k][nb][pb], 0, 0, 0);
      }
    };
    if (c0 < c1) {
      load(0, c0);
      for (int c = c0; c < c1; c += 2 * SU) {
        load(1, c + SU < c1 ? c + SU : c1 - 1);
        mul(0, c);
        if (c + SU >= c1) break;
        load(0, c + 2 * SU < c1 ? c + 2 * SU : c1 - 1);
        mul(1, c + SU);
      }
    }
  }
  // sums over the waves, one stream after the other
  const int row = tid >> 3, cq = 4 * (tid & 7);     // threads 0..255: point, first column
  float v[C][4];
#pragma unroll
  for (int k = 0; k < C; ++k) {
    double* pw = part[wave];
    if (k > 0) __syncthreads();                      // the previous stream has been summed
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          pw[(16 * pb + (lane & 15)) * PITCH + 16 * nb + (lane >> 4) + 4 * r] = accd[k][nb][pb][r];
    __syncthreads();
    if (tid < 256) {
      double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] += part[w][row * PITCH + cq + e];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[k][e] = (float)t[e];
    }
  }
  const int64_t pt = m0 + row;
  if (tid >= 256 || pt >= npts) return;
  const int n = n0 + cq;
  if constexpr (EPI == EPI_DF) {
    const int64_t ldY = p.sY_ld > 0 ? p.sY_ld : p.nY, ldU = p.sU_ld > 0 ? p.sU_ld : p.nU;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float o = p.df_sign * v[0][e];
      if (n + e < p.nY) p.seedY[g * p.sY_g + pt * ldY + n + e] = o;
      else if (n + e < p.nY + p.nU) p.seedU[g * p.sU_g + pt * ldU + p.sU_off + (n + e - p.nY)] = o;
    }
    return;
  } else {
    auto at = [&](auto* base, int k) { return base + g * p.o_g + (p.seg.row0 + k * p.seg.plane + pt) * p.ldo + n; };
    auto put = [&](float* dst) {
#pragma unroll
      for (int k = 0; k < C; ++k) store4<float>(at(dst, k), v[k]);
    };
    auto add = [&](const float* src) {
#pragma unroll
      for (int k = 0; k < C; ++k) {
        float s4[4];
        load4<float>(at(src, k), s4);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[k][e] += s4[e];
      }
    };
    if constexpr (EPI == EPI_FWD) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[0][e] += p.bias[g * p.b_g + n + e];
      if (p.out_a) put(p.out_a);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float x[C];
#pragma unroll
        for (int k = 0; k < C; ++k) x[k] = v[k][e];
        jet_fwd<ND1, 0, true>(x);
#pragma unroll
        for (int k = 0; k < C; ++k) v[k][e] = x[k];
      }
      if (p.skip) add(p.skip);
      put(p.out_h);
    } else {
      if (p.skip_g) add(p.skip_g);
      if (p.out_gh) put(p.out_gh);
      float ap[C][4];
#pragma unroll
      for (int k = 0; k < C; ++k) load4<float>(at(p.aprev, k), ap[k]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float gv[C], av[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
          gv[k] = v[k][e];
          av[k] = ap[k][e];
        }
        jet_bwd<ND1, 0, true>(gv, av);
#pragma unroll
        for (int k = 0; k < C; ++k) v[k][e] = gv[k];
      }
      put(p.out_da);
    }
  }
}

// ---------------------------------------------------------------------------
// k_gemm_short_x2: the split products (PM_SPLIT2) of k_gemm_nt where a launch
// has few output tiles.  One wave per 32 points x 32 columns walks the
// contraction in k_gemm_nt's order (so the results are the same bits), with
// SU 16-wide chunks of operands in registers and as many on their way: no LDS,
// no barrier, and 32 times as many waves in flight as blocks of the 64 x 256
// tile.
// ---------------------------------------------------------------------------
template <int ND1, int EPI>
__global__ void __launch_bounds__(64) k_gemm_short_x2(const NtArgs<float> p) {
  constexpr int C = 1 + ND1;
  constexpr int SU = C == 1 ? 8 : 5;
  const int g = blockIdx.z;
  const int lane = threadIdx.x;
  const int hh = lane >> 5;
  const int ntn = p.N / 32;
  const int64_t lt = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t m0 = (lt / ntn) * 32;
  const int n0 = (int)(lt % ntn) * 32;
  const int64_t npts = p.seg.n_points;
  const int nch = p.K / 16;
  const bool pvalid = m0 + (lane & 31) < npts;
  // points past the end read the last one (their results are never stored)
  const int64_t pt = pvalid ? m0 + (lane & 31) : npts - 1;
  // lane: row l & 31, eight k values 8 (l >> 5) of a chunk; the weight rows
  // hold a chunk's 16 high pieces, then its 16 low pieces
  const char* wp = (const char*)(p.Wm + g * p.w_g + (int64_t)(n0 + (lane & 31)) * p.ldw) + 16 * hh;
  const char* xp[C];
#pragma unroll
  for (int k = 0; k < C; ++k)
    xp[k] = (const char*)(p.X + g * p.x_g + (p.seg.row0 + k * p.seg.plane + pt) * p.ldx) + 32 * hh;
  f32x16 acc[C];
#pragma unroll
  for (int k = 0; k < C; ++k)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[k][r] = 0.0f;
  u32x4 wb[2][SU][2], xb[2][SU][C][2];
  auto load = [&](int b, int c) {
#pragma unroll
    for (int i = 0; i < SU; ++i) {
      const int64_t o = (int64_t)(c + i < nch ? c + i : nch - 1) * 64;   // (repeats of the last chunk are not multiplied)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        wb[b][i][h] = *(const u32x4*)(wp + o + 32 * h);
#pragma unroll
        for (int k = 0; k < C; ++k) xb[b][i][k][h] = *(const u32x4*)(xp[k] + o + 16 * h);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mul = [&](int b, int c) {
#pragma unroll
    for (int i = 0; i < SU; ++i) {
      if (c + i >= nch) break;
      const bf16x8 bw[2] = {__builtin_bit_cast(bf16x8, wb[b][i][0]), __builtin_bit_cast(bf16x8, wb[b][i][1])};
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const u32x8 w = {xb[b][i][k][0].x, xb[b][i][k][0].y, xb[b][i][k][0].z, xb[b][i][k][0].w,
                         xb[b][i][k][1].x, xb[b][i][k][1].y, xb[b][i][k][1].z, xb[b][i][k][1].w};
        bf16x8 ax[2];
        split_frag(__builtin_bit_cast(f32x8, w), ax);
        mma_split(acc[k], bw, ax);
      }
    }
  };
  load(0, 0);
  for (int c = 0; c < nch; c += 2 * SU) {
    load(1, c + SU);
    mul(0, c);
    if (c + SU >= nch) break;
    load(0, c + 2 * SU);
    mul(1, c + SU);
  }

  // lane: point pt, columns n0 + 8 q + 4 hh + 0..3 in registers 4 q + 0..3
  if constexpr (EPI == EPI_DF) {
    const int64_t ldY = p.sY_ld > 0 ? p.sY_ld : p.nY, ldU = p.sU_ld > 0 ? p.sU_ld : p.nU;
    if (!pvalid) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int n = n0 + 8 * (r >> 2) + 4 * hh + (r & 3);
      const float v = p.df_sign * acc[0][r];
      if (n < p.nY) p.seedY[g * p.sY_g + pt * ldY + n] = v;
      else if (n < p.nY + p.nU) p.seedU[g * p.sU_g + pt * ldU + p.sU_off + (n - p.nY)] = v;
    }
  } else {
    auto at = [&](auto* base, int k, int q) {
      return base + g * p.o_g + (p.seg.row0 + k * p.seg.plane + pt) * p.ldo + n0 + 8 * q + 4 * hh;
    };
    auto put = [&](float* dst) {
      if (!pvalid) return;
#pragma unroll
      for (int k = 0; k < C; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(f32x4*)at(dst, k, q) = f32x4{acc[k][4 * q], acc[k][4 * q + 1], acc[k][4 * q + 2], acc[k][4 * q + 3]};
    };
    auto get = [&](f32x4 (&v)[C][4], const float* src) {
#pragma unroll
      for (int k = 0; k < C; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) v[k][q] = *(const f32x4*)at(src, k, q);
    };
    auto add = [&](const float* src) {
      f32x4 v[C][4];
      get(v, src);
#pragma unroll
      for (int k = 0; k < C; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] += v[k][r >> 2][r & 3];
    };
    if constexpr (EPI == EPI_FWD) {
      const float* bp = p.bias + g * p.b_g + n0 + 4 * hh;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][r] += bp[8 * (r >> 2) + (r & 3)];
      if (p.out_a) put(p.out_a);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v[C];
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = acc[k][r];
        jet_fwd<ND1, 0>(v);
#pragma unroll
        for (int k = 0; k < C; ++k) acc[k][r] = v[k];
      }
      if (p.skip) add(p.skip);
      put(p.out_h);
    } else {
      f32x4 ap[C][4];
      get(ap, p.aprev);
      if (p.skip_g) add(p.skip_g);
      if (p.out_gh) put(p.out_gh);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float gv[C], av[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
          gv[k] = acc[k][r];
          av[k] = ap[k][r >> 2][r & 3];
        }
        jet_bwd<ND1, 0>(gv, av);
#pragma unroll
        for (int k = 0; k < C; ++k) acc[k][r] = gv[k];
      }
      put(p.out_da);
    }
  }
}

// ---------------------------------------------------------------------------
// k_gemm_nt_wr: the products and epilogues of k_gemm_nt for 16-bit storage
// and K = N = 128 (hidden layers of width 128), as a persistent kernel
// built to keep HBM busy.  Each block copies the weight matrix into LDS once
// and then walks tiles of 32 points (all jet streams, the whole K extent at
// once).  While one tile is multiplied and written out, the activations of
// its successor (and, in the reverse pass, the saved pre-activations of the
// tile itself) are already on their way into registers, so every block keeps
// a whole tile of loads in flight.  Four waves; wave w owns columns
// 32w..32w+31 of every stream.  SKIP: the residual blocks of a shared trunk
// (forward: h_l += h_{l-2}; reverse: the block's skip cotangent added, the
// total kept), read like the saved pre-activations, ahead of the prefetch.
// ---------------------------------------------------------------------------
// one block per CU (and the whole register file) for the skip variant of
// five streams, whose skip rows do not fit beside the prefetch otherwise
template <int C, bool SKIP, bool TWO = false>
constexpr int wr_blocks_per_cu() { return (SKIP || TWO) && C >= 5 ? 1 : 2; }

// TWO: two-term weight rows [W_hi | W_lo] (forward, K = 2 x 128): W_hi is the
// LDS-resident tile, each wave keeps its columns' W_lo fragments in registers
// for the whole launch.
template <class T, int ND1, int ND2, int EPI, bool FIRST, bool SKIP = false, bool TWO = false>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(wr_blocks_per_cu<1 + ND1 + ND2, SKIP, TWO>())))
k_gemm_nt_wr(const NtArgs<T> p, int64_t ntiles) {
  static_assert(sizeof(T) == 2, "16-bit storage only");
  static_assert(!(SKIP && FIRST), "residual blocks never start at the first layer");
  static_assert(!TWO || EPI == EPI_FWD, "two-term weights: forward products only");
  constexpr int C = 1 + ND1 + ND2;
  constexpr int BM = 32, BN = 128, NTH = 256, ES = 2;
  constexpr int RB = 256;                          // bytes of one operand row (K = 128)
  constexpr int PITCH = RB + 16;                   // LDS row pitch: conflict-free 16-byte fragment reads
  constexpr int WREG = BN * PITCH;                 // weight tile
  constexpr int XREG = C * BM * PITCH;             // activation tile, reused to stage the outputs
  constexpr int OPITCH = BN * ES + 16;             // staging pitch of one output plane
  static_assert(C * BM * OPITCH <= XREG, "staging must fit in the activation region");
  constexpr int SEGS = RB / 16;                    // 16-byte pieces per row
  constexpr int XP = C * BM * SEGS / NTH;          // pieces per thread of an activation tile
  constexpr int WP = BN * SEGS / NTH;              // pieces per thread of the weights
  constexpr int RPP = NTH / SEGS;                  // rows covered by one piece index
  typedef typename Elem<T>::frag frag;
  constexpr int W1REG = FIRST ? BN * 4 * 4 : 0;   // W1 columns 0..2 of every unit (fp32, padded to 4)
  __shared__ __attribute__((aligned(16))) char lds[WREG + XREG + W1REG];
  char* const wl = lds;
  char* const xl = lds + WREG;
  float* const w1l = (float*)(lds + WREG + XREG);

  const int g = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int hh = lane >> 5;
  const int sg = tid % SEGS;
  const int64_t npts = p.seg.n_points;
  const char* Xb = (const char*)(p.X + g * p.x_g);
  const char* Wb = (const char*)(p.Wm + g * p.w_g);

  // weights (N = 128 rows)
  {
    u32x4 wb[WP];
#pragma unroll
    for (int i = 0; i < WP; ++i) wb[i] = *(const u32x4*)(Wb + (int64_t)(tid / SEGS + RPP * i) * p.ldw * ES + sg * 16);
#pragma unroll
    for (int i = 0; i < WP; ++i) *(u32x4*)(wl + (tid / SEGS + RPP * i) * PITCH + sg * 16) = wb[i];
  }
  // the low terms of the wave's 32 weight rows, one fragment per 16-wide k chunk
  frag wlo[TWO ? RB / 32 : 1];
  if constexpr (TWO) {
    const char* wrow = Wb + (int64_t)(32 * wave + (lane & 31)) * p.ldw * ES + RB;
#pragma unroll
    for (int c = 0; c < RB / 32; ++c) wlo[c] = *(const frag*)(wrow + c * 32 + hh * 16);
  }

  // first layer formed in the kernel: W1[n][0..d-1] for every unit n
  if constexpr (FIRST) {
    if (tid < BN) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w1l[tid * 4 + i] = i < p.f_d ? p.fp1[g * p.fp_g + (int64_t)tid * p.f_in + i] : 0.0f;
    }
    lds_sync();
  }
  // sample and coordinate row of point pt of the segment
  auto f_sample = [&](int64_t pt) { return pt / p.fPn; };
  auto f_xrow = [&](int64_t pt) { return p.fx_shared ? pt % p.fPn : pt; };

  // activation rows of a tile; points past the end repeat the last point.
  // Stream bases are uniform (scalar); a thread's two point rows are 32-bit
  // byte offsets (the host checks that a stream plane spans < 2^31 bytes).
  static_assert(BM == 2 * RPP, "two point rows per thread");
  constexpr bool GENX = FIRST && EPI == EPI_FWD;   // forward: X is the first layer's activations
  constexpr int XPR = GENX ? 1 : XP;
  u32x4 xb[XPR];
  // first layer: the thread's two points (rows tid / SEGS + RPP j) and its 8
  // units 8 sg..8 sg+7: coordinates and z-projection of the next tile
  float fxv[2][3], fzv[2][8];
  auto xload = [&](int64_t tile) {
    int64_t p0 = tile * BM + tid / SEGS, p1 = p0 + RPP;
    if (p0 >= npts) p0 = npts - 1;
    if (p1 >= npts) p1 = npts - 1;
    if constexpr (GENX) {
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int64_t pt = jj ? p1 : p0;
        const float* xv = p.fx + g * p.fx_g + f_xrow(pt) * p.f_d;
#pragma unroll
        for (int i = 0; i < 3; ++i) fxv[jj][i] = i < p.f_d ? xv[i] : 0.0f;
        const float4* zv = (const float4*)(p.fzp + g * p.fzp_g + f_sample(pt) * BN + 8 * sg);
        const float4 z0 = zv[0], z1 = zv[1];
        fzv[jj][0] = z0.x; fzv[jj][1] = z0.y; fzv[jj][2] = z0.z; fzv[jj][3] = z0.w;
        fzv[jj][4] = z1.x; fzv[jj][5] = z1.y; fzv[jj][6] = z1.z; fzv[jj][7] = z1.w;
      }
    } else {
      const uint32_t o0 = (uint32_t)(p0 * p.ldx * ES) + sg * 16, o1 = (uint32_t)(p1 * p.ldx * ES) + sg * 16;
#pragma unroll
      for (int i = 0; i < XP; ++i) {
        const char* base = Xb + (p.seg.row0 + (i >> 1) * p.seg.plane) * p.ldx * ES;
        xb[i] = *(const u32x4*)(base + ((i & 1) ? o1 : o0));
      }
    }
  };
  auto ncol = [&](int q) { return 32 * wave + 8 * q + 4 * hh; };   // first of the lane's 4 columns in group q

  // bias and output weights of the lane's 16 columns (fixed for the launch)
  float bias[16], wo[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) bias[r] = wo[r] = 0.0f;
  float bout = 0.0f;
  if (EPI == EPI_FWD && p.bias) {
#pragma unroll
    for (int r = 0; r < 16; ++r) bias[r] = p.bias[g * p.b_g + ncol(r >> 2) + (r & 3)];
  }
  if (!SKIP && EPI == EPI_FWD && p.y) {           // (the output layer is never fused with a skip)
#pragma unroll
    for (int r = 0; r < 16; ++r) wo[r] = p.wout[g * p.wo_g + ncol(r >> 2) + (r & 3)];
    bout = p.wout[g * p.wo_g + BN];
  }

  auto pack8 = [&](const float* v) {
    u32x4 w;
#pragma unroll
    for (int h2 = 0; h2 < 4; ++h2) {
      const T lo = Elem<T>::from_f(v[2 * h2]), hi = Elem<T>::from_f(v[2 * h2 + 1]);
      w[h2] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
    return w;
  };
  auto xstore = [&](int64_t tile) {
    if constexpr (GENX) {
      // first layer, as in the standalone kernel: a = zproj + sum_i W1[:, i] x_i,
      // h = t, h'_i = s W1[:, i], h''_i = s' W1[:, i]^2 (a' = W1[:, i], a'' = 0)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        int64_t pt = tile * BM + tid / SEGS + RPP * jj;
        if (pt >= npts) pt = npts - 1;
        float a[8], hv[8], s8[8], sp8[8], fwc[3][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float4 w4 = *(const float4*)(w1l + (8 * sg + e) * 4);
          fwc[0][e] = w4.x; fwc[1][e] = w4.y; fwc[2][e] = w4.z;
          a[e] = fzv[jj][e];
#pragma unroll
          for (int i = 0; i < 3; ++i) a[e] += fwc[i][e] * fxv[jj][i];
          float t, sd;
          tanh_ts(a[e], t, sd);
          hv[e] = t;
          s8[e] = sd;
          sp8[e] = -2.0f * t * sd;
        }
        const int row = tid / SEGS + RPP * jj;
#pragma unroll
        for (int k = 0; k < C; ++k) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            if (k == 0) v[e] = hv[e];
            else if (k <= ND1) v[e] = s8[e] * fwc[k - 1][e];
            else v[e] = sp8[e] * fwc[k - 1 - ND1][e] * fwc[k - 1 - ND1][e];
          }
          const u32x4 w = pack8(v);
          *(u32x4*)(xl + (k * BM + row) * PITCH + sg * 16) = w;
          if (p.f_out_h)                           // past the end: the last point's values again
            *(u32x4*)(p.f_out_h + g * p.o_g + (p.seg.row0 + k * p.seg.plane + pt) * p.ldo + 8 * sg) = w;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < XP; ++i) *(u32x4*)(xl + (tid / SEGS + RPP * i) * PITCH + sg * 16) = xb[i];
    }
  };

  // The activations of a tile go from registers to LDS at the end of the
  // previous iteration, after its stores were issued: the wait for the
  // prefetch then leaves those stores in flight (the memory counter drains
  // in issue order, and the same operations are pending on every iteration).
  int64_t tile = blockIdx.x;
  xload(tile);
  xstore(tile);
  for (; tile < ntiles; tile += gridDim.x) {
    const int64_t m0 = tile * BM;
    lds_sync();

    // reverse pass: the saved pre-activations of this tile, in the lane
    // layout of the products (point lane & 31, four columns per group).
    // Issued before the prefetch so that waiting for them (the memory
    // counter drains in issue order) does not wait for the prefetch.
    u32x2 apr[FIRST ? 1 : C][4];
    float fzb[16], fxb[3];
    if (FIRST && EPI == EPI_BWD) {
      // first layer: z-projection of the lane's 16 units and its coordinates
      int64_t pt = m0 + (lane & 31);
      if (pt >= npts) pt = npts - 1;
      const float* zr = p.fzp + g * p.fzp_g + f_sample(pt) * BN;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 z4 = *(const float4*)(zr + ncol(q));
        fzb[4 * q] = z4.x; fzb[4 * q + 1] = z4.y; fzb[4 * q + 2] = z4.z; fzb[4 * q + 3] = z4.w;
      }
      const float* xv = p.fx + g * p.fx_g + f_xrow(pt) * p.f_d;
#pragma unroll
      for (int i = 0; i < 3; ++i) fxb[i] = i < p.f_d ? xv[i] : 0.0f;
    } else if (EPI == EPI_BWD) {
      int64_t pt = m0 + (lane & 31);
      if (pt >= npts) pt = npts - 1;
      const uint32_t po = (uint32_t)(pt * p.ldo * ES);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const bool one_row = SKIP && k > 0 && p.a_seeds;   // (launches without a skip have whole streams)
        const char* base = (const char*)(p.aprev + g * p.o_g +
                                         (p.seg.row0 + (one_row ? p.seg.plane + k - 1 : k * p.seg.plane)) * p.ldo);
        const uint32_t pk = one_row ? 0u : po;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          apr[k][q] = *(const u32x2*)(base + pk + ncol(q) * ES);
        }
      }
    }
    // residual skip of the tile in the same lane layout: the block input
    // h_{l-2} (forward) or the skip cotangent of a block input (reverse)
    u32x2 skp[SKIP ? C : 1][4];
    const T* const skip_src = EPI == EPI_FWD ? p.skip : p.skip_g;
    if (SKIP && skip_src) {
      int64_t pt = m0 + (lane & 31);
      if (pt >= npts) pt = npts - 1;
      const uint32_t po = (uint32_t)(pt * p.ldo * ES);
#pragma unroll
      for (int k = 0; k < (SKIP ? C : 1); ++k) {
        const char* base = (const char*)(skip_src + g * p.o_g + (p.seg.row0 + k * p.seg.plane) * p.ldo);
#pragma unroll
        for (int q = 0; q < 4; ++q) skp[k][q] = *(const u32x2*)(base + po + ncol(q) * ES);
      }
    }

    {
      const int64_t nx = tile + gridDim.x;
      xload(nx < ntiles ? nx : tile);              // unconditional: the last prefetch is never used
    }
    __builtin_amdgcn_sched_barrier(0);             // keep the loads ahead of the products

    f32x16 acc[C];
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[k][r] = 0.0f;
    // register r of a lane holds column ncol(r / 4) + r % 4 of its point,
    // which is element r % 4 of the lane's u32x2 pair (r / 4)
    auto add_skip = [&]() {
#pragma unroll
      for (int k = 0; k < (SKIP ? C : 1); ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const uint32_t w = skp[k][r >> 2][(r & 3) >> 1];
          const uint16_t h = (r & 1) ? (uint16_t)(w >> 16) : (uint16_t)(w & 0xffffu);
          acc[k][r] += Elem<T>::to_f(__builtin_bit_cast(T, h));
        }
    };
#pragma unroll
    for (int c = 0; c < RB / 32; ++c) {
      const int koff = c * 32 + hh * 16;
      const frag bfr = *(const frag*)(wl + (32 * wave + (lane & 31)) * PITCH + koff);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const frag afr = *(const frag*)(xl + (k * BM + (lane & 31)) * PITCH + koff);
        if constexpr (TWO) Elem<T>::mma(acc[k], wlo[c], afr);
        Elem<T>::mma(acc[k], bfr, afr);            // rows: columns n; cols: points
      }
    }
    __builtin_amdgcn_sched_barrier(0);             // no epilogue work (waits on the loads) above here
    lds_sync();                                    // the activation region is free for staging

    // all C output planes of the tile at once: stream k is staged in rows
    // [32k, 32k+32) of the (free) activation region, then copied out in
    // full 16-byte row segments
    auto stage_out = [&](T* dst) {
#pragma unroll
      for (int k = 0; k < C; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[k][4 * q + e];
          store4<T>((T*)(xl + (k * BM + (lane & 31)) * OPITCH + ncol(q) * ES), v);
        }
      lds_sync();
      // rows of points past the end hold exactly the values of the last
      // point (same inputs, same arithmetic): they are written over it
      // unconditionally, which keeps the memory counter static for the
      // prefetch waits
      constexpr int CPR = BN * ES / 16;            // 16-byte chunks per row
#pragma unroll
      for (int j = 0; j < C * BM * CPR / NTH; ++j) {
        const int i = tid + j * NTH;
        const int row = i / CPR, ch = i % CPR;
        const int k = row / BM;
        int64_t pt = m0 + row % BM;
        if (pt >= npts) pt = npts - 1;
        *(u32x4*)(dst + g * p.o_g + (p.seg.row0 + k * p.seg.plane + pt) * p.ldo + ch * (16 / ES)) =
            *(const u32x4*)(xl + row * OPITCH + ch * 16);
      }
      lds_sync();
    };

    if (EPI == EPI_FWD) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][r] += bias[r];
      if (p.out_a) {
        stage_out(p.out_a);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v[C];
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = acc[k][r];
        jet_fwd<ND1, ND2>(v);
#pragma unroll
        for (int k = 0; k < C; ++k) acc[k][r] = v[k];
      }
      if constexpr (SKIP) {
        if (p.skip) add_skip();                    // residual block output
      }
      if (!SKIP && p.y) {
        // output layer: y = w_out . h over the activations as stored, summed
        // over the lane's columns, the two lane halves, then the four waves
        // in wave order (through LDS)
        float* red = (float*)xl;
#pragma unroll
        for (int k = 0; k < C; ++k) {
          float part = 0.0f;
#pragma unroll
          for (int r = 0; r < 16; ++r) part += wo[r] * Elem<T>::to_f(Elem<T>::from_f(acc[k][r]));
          part += __shfl_xor(part, 32);
          if (lane < 32) red[(wave * C + k) * 32 + lane] = part;
        }
        lds_sync();
        if (tid < C * 32) {
          const int k = tid >> 5, pp = tid & 31;
          float v = red[k * 32 + pp];
#pragma unroll
          for (int w = 1; w < 4; ++w) v += red[(w * C + k) * 32 + pp];
          if (k == 0) v += bout;
          int64_t pt = m0 + pp;
          if (pt >= npts) pt = npts - 1;             // past the end: the last point's value again
          p.y[g * p.y_g + p.seg.row0 + k * p.seg.plane + pt] = v;
        }
        lds_sync();
      }
      if (p.out_h) stage_out(p.out_h);
    } else {
      if constexpr (SKIP) {
        // skip cotangent of a residual block's input, and the total kept for
        // the skip below it (all loads of the tile were consumed before the
        // staging barrier, so an in-place total is safe)
        if (p.skip_g) add_skip();
        if (p.out_gh) stage_out(p.out_gh);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * q + e;
          float gv[C], av[C];
#pragma unroll
          for (int k = 0; k < C; ++k) gv[k] = acc[k][r];
          if constexpr (FIRST) {
            // the first layer's pre-activations as the standalone pass stores
            // them: a (rounded), a'_i = W1[n][i] (rounded), a''_i = 0
            const float* w1 = w1l + (ncol(q) + e) * 4;
            float a = fzb[r];
#pragma unroll
            for (int i = 0; i < 3; ++i) a += w1[i] * fxb[i];
            av[0] = Elem<T>::to_f(Elem<T>::from_f(a));
#pragma unroll
            for (int i = 0; i < ND1; ++i) av[1 + i] = Elem<T>::to_f(Elem<T>::from_f(w1[i]));
#pragma unroll
            for (int i = 0; i < ND2; ++i) av[1 + ND1 + i] = 0.0f;
          } else {
#pragma unroll
            for (int k = 0; k < C; ++k) {
              const uint32_t w = apr[k][q][e >> 1];
              const uint16_t h = (e & 1) ? (uint16_t)(w >> 16) : (uint16_t)(w & 0xffffu);
              av[k] = Elem<T>::to_f(__builtin_bit_cast(T, h));
            }
          }
          jet_bwd<ND1, ND2>(gv, av);
#pragma unroll
          for (int k = 0; k < C; ++k) acc[k][r] = gv[k];
        }
      }
      stage_out(p.out_da);
    }
    {
      const int64_t nx = tile + gridDim.x;
      xstore(nx < ntiles ? nx : tile);             // the next tile (the region is free again)
    }
  }
}

// ---------------------------------------------------------------------------
// dW[n][j] = sum_{rows m} dA[m][n] H[m][j]   (contraction over rows)
// Each block owns a (BNn x BJ) output tile and one contiguous range of rows.
// Row slices are transposed into LDS: every operand column is one 64-byte
// line of SR rows (8 rows per 16-byte fragment), so the fragments are single
// 16-byte reads.  Line base of column c (bytes): 80 c, plus 64 for columns
// 16..31 of every 32 (period 2624 bytes).  With lanes running over 16 row
// pairs x 4 column groups, each transposing write instruction then hits 64
// distinct banks, and the fragment reads stay conflict-free.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int dw_col(int c) {
  return (c >> 5) * 2624 + (c & 31) * 80 + ((c & 16) ? 64 : 0);
}

// PM (fp32 storage): how the products are formed (ProdMode); with PM_F64 the
// split partials are written in fp64 to partial64 (partial is unused).
template <class T, int WM, int WN, int NT, int OCC, int NB, int PM = PM_NATIVE>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC)))
k_gemm_dw(const T* __restrict__ dA, int64_t a_g, int64_t lda, const T* __restrict__ H, int64_t h_g,
          int64_t ldh, int64_t R, int64_t n_value, int N, int J, float* __restrict__ partial,
          double* __restrict__ pdb, int n_split, int64_t rows_per_split, double* __restrict__ partial64) {
  static_assert(PM == PM_NATIVE || sizeof(T) == 4, "split products: fp32 storage");
  constexpr int BNn = 32 * NT * WM;
  constexpr int BJ = 32 * NT * WN;
  constexpr int NTH = 64 * WM * WN;
  constexpr int ES = (int)sizeof(T);
  constexpr int SR = 64 / ES;               // rows per stage
  constexpr int EPP = 16 / ES;              // elements per 16-byte load
  // PM_SPLIT2: every fp32 value is cut into its two bf16 pieces once, as the
  // stage is stored; a 64-byte column line (16 rows) then holds the 16 high
  // pieces followed by the 16 low pieces
  constexpr bool SPL = PM == PM_SPLIT2;
  constexpr int RPP = (ES == 2 || SPL) ? 2 : 1;   // rows per piece (packed 4-byte LDS writes)
  constexpr int NRP = SR / RPP;             // row pieces per stage (16)
  constexpr int NCH = 64 / (16 * ES);
  constexpr int PA = NRP * (BNn / EPP);
  constexpr int PB = NRP * (BJ / EPP);
  constexpr int PIECES = PA + PB;
  constexpr int PPT = (PIECES + NTH - 1) / NTH;
  constexpr int REGA = (BNn / 32) * 2624;   // bytes of the dA part of a stage
  constexpr int STAGE = REGA + (BJ / 32) * 2624;
  typedef typename Elem<T>::frag frag;
  __shared__ __attribute__((aligned(16))) char lds[2 * STAGE];

  // logical block: output tiles fastest, so the blocks reading one row range
  // run together on one XCD
  const int tiles_n = (N + BNn - 1) / BNn;
  const int tiles = tiles_n * ((J + BJ - 1) / BJ);
  const int64_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = (int)(lb % tiles);
  const int tn = tile % tiles_n;
  const int tj = tile / tiles_n;
  const int split = (int)(lb / tiles);
  const int g = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % WM;
  const int wn = wave / WM;
  const int n0 = tn * BNn;
  const int j0 = tj * BJ;
  const int64_t r0 = (int64_t)split * rows_per_split;
  const int64_t r1 = r0 + rows_per_split < R ? r0 + rows_per_split : R;
  const int64_t rv = r1 < n_value ? r1 : n_value;
  const int nst = (int)((r1 - r0 + SR - 1) / SR);

  const T* A = dA + g * a_g;
  const T* B = H + g * h_g;

  f32x16 acc[NT][NT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
  // PM_F64: a wave's 32 x 32 outputs as 2 x 2 blocks of the 16 x 16 fp64
  // product (lane l: rows (l >> 4) + 4 r, column l & 15 of a block)
  static_assert(PM != PM_F64 || NT == 1, "fp64 products: one fragment per wave");
  f64x4 accd[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) accd[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  double dbacc = 0.0;

  // piece q of an operand: row piece q % NRP, column group q / NRP
  auto gload = [&](uint4 (*buf)[RPP], int64_t k0) {
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int piece = tid + i * NTH;
      const bool isA = piece < PA;
      const int q = isA ? piece : piece - PA;
      const int rp = q % NRP, cg = q / NRP;
      const int col = (isA ? n0 : j0) + cg * EPP;
      const int lim = isA ? N : J;
      // rows past the split range load a clamped row (zeroed when stored to
      // LDS); columns past the end only reach outputs that are never stored
      const int colc = col < lim ? col : lim - EPP;
#pragma unroll
      for (int u = 0; u < RPP; ++u) {
        const int64_t row = k0 + rp * RPP + u;
        const int64_t rowc = row < r1 ? row : r1 - 1;
        buf[i][u] = isA ? *(const uint4*)(A + rowc * lda + colc) : *(const uint4*)(B + rowc * ldh + colc);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // keep the prefetch where it is issued
  };
  auto lstore = [&](const uint4 (*buf)[RPP], int stage, int64_t k0) {
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int piece = tid + i * NTH;
      if (piece >= PIECES) continue;
      const bool isA = piece < PA;
      const int q = isA ? piece : piece - PA;
      const int rp = q % NRP, cg = q / NRP;
      char* base = lds + stage * STAGE + (isA ? 0 : REGA);
      const uint32_t m0k = (k0 + rp * RPP < r1) ? 0xffffffffu : 0u;            // row validity masks
      const uint32_t m1k = (k0 + rp * RPP + RPP - 1 < r1) ? 0xffffffffu : 0u;
      if constexpr (SPL) {
        // rows 2 rp and 2 rp + 1: one word of high pieces, one of low pieces
        const float* x0 = (const float*)&buf[i][0];
        const float* x1 = (const float*)&buf[i][RPP - 1];
#pragma unroll
        for (int e = 0; e < EPP; ++e) {
          const bf16 h0 = (bf16)x0[e], h1 = (bf16)x1[e];
          const bf16 l0 = (bf16)(x0[e] - (float)h0), l1 = (bf16)(x1[e] - (float)h1);
          char* line = base + dw_col(cg * EPP + e) + rp * 4;
          *(uint32_t*)line = ((uint32_t)__builtin_bit_cast(uint16_t, h0) & m0k & 0xffffu) |
                             (((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16) & m1k);
          *(uint32_t*)(line + 32) = ((uint32_t)__builtin_bit_cast(uint16_t, l0) & m0k & 0xffffu) |
                                    (((uint32_t)__builtin_bit_cast(uint16_t, l1) << 16) & m1k);
        }
      } else if (ES == 2) {
        const uint16_t* lo = (const uint16_t*)&buf[i][0];
        const uint16_t* hi = (const uint16_t*)&buf[i][RPP - 1];
#pragma unroll
        for (int e = 0; e < EPP; ++e)
          *(uint32_t*)(base + dw_col(cg * EPP + e) + rp * 4) =
              ((uint32_t)lo[e] & m0k & 0xffffu) | (((uint32_t)hi[e] << 16) & m1k);
      } else {
        const uint32_t* v = (const uint32_t*)&buf[i][0];
#pragma unroll
        for (int e = 0; e < EPP; ++e) *(uint32_t*)(base + dw_col(cg * EPP + e) + rp * 4) = v[e] & m0k;
      }
    }
  };
  auto compute = [&](int stage, int64_t k0) {
    const char* base = lds + stage * STAGE;
    if constexpr (PM == PM_F64) {
      // fp32 rows of each column line, four at a time through the fp64 product
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const int ro = (4 * kk + (lane >> 4)) * 4;
        double av[2], bv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          av[h] = (double)*(const float*)(base + dw_col(32 * wm + 16 * h + (lane & 15)) + ro);
          bv[h] = (double)*(const float*)(base + REGA + dw_col(32 * wn + 16 * h + (lane & 15)) + ro);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b) accd[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], accd[a][b], 0, 0, 0);
      }
    }
    if constexpr (SPL) {
      // high pieces at byte 0 of a column line, low pieces at byte 32
      const int koff = (lane >> 5) * 16;
      bf16x8 ap[NT][2], bp[NT][2];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          ap[t][c] = *(const bf16x8*)(base + dw_col(32 * (wm * NT + t) + (lane & 31)) + 32 * c + koff);
          bp[t][c] = *(const bf16x8*)(base + REGA + dw_col(32 * (wn * NT + t) + (lane & 31)) + 32 * c + koff);
        }
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) mma_split(acc[a][b], ap[a], bp[b]);
    }
#pragma unroll
    for (int c = 0; c < (PM == PM_F64 || SPL ? 0 : NCH); ++c) {
      const int koff = c * 32 + (lane >> 5) * (8 * ES);
      frag af[NT], bf[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        af[t] = *(const frag*)(base + dw_col(32 * (wm * NT + t) + (lane & 31)) + koff);
        bf[t] = *(const frag*)(base + REGA + dw_col(32 * (wn * NT + t) + (lane & 31)) + koff);
      }
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) Elem<T>::mma(acc[a][b], af[a], bf[b]);
    }
    // bias cotangent: value rows of this slice, one column per thread
    // (the 64-byte column line is read as 16 independent words)
    if (pdb && tj == 0 && tid < BNn && k0 < rv) {
      const int nr = (int)((rv - k0) < SR ? (rv - k0) : SR);
      const uint32_t* colw = (const uint32_t*)(base + dw_col(tid));
      typename std::conditional<ES == 4, double, float>::type part_sum = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        const uint32_t v = colw[w];
        if constexpr (SPL) {
          // words 0-7: high pieces of rows 2w, 2w + 1; words 8-15: low pieces
          if (w < 8) {
            const uint32_t l = colw[w + 8];
            const double r0 = (double)(float)__builtin_bit_cast(bf16, (uint16_t)(v & 0xffffu)) +
                              (double)(float)__builtin_bit_cast(bf16, (uint16_t)(l & 0xffffu));
            const double r1 = (double)(float)__builtin_bit_cast(bf16, (uint16_t)(v >> 16)) +
                              (double)(float)__builtin_bit_cast(bf16, (uint16_t)(l >> 16));
            part_sum += (2 * w < nr ? r0 : 0.0) + (2 * w + 1 < nr ? r1 : 0.0);
          }
        } else if constexpr (ES == 2) {
          const float lo = Elem<T>::to_f(__builtin_bit_cast(T, (uint16_t)(v & 0xffffu)));
          const float hi = Elem<T>::to_f(__builtin_bit_cast(T, (uint16_t)(v >> 16)));
          part_sum += (2 * w < nr ? lo : 0.0f) + (2 * w + 1 < nr ? hi : 0.0f);
        } else {
          part_sum += w < nr ? (double)__uint_as_float(v) : 0.0;
        }
      }
      dbacc += (double)part_sum;
    }
  };

  if constexpr (OCC >= 2 || NB > 2) {
    // two LDS stages and a ring of NB register buffers: buffer b holds the
    // stages s = b (mod NB), so NB stages of loads are in flight while one is
    // multiplied.  Loads are unconditional (stage index clamped, rows past
    // the range zeroed at the LDS store), so the waits are static counts.
    uint4 bufs[NB][PPT][RPP];
    const int last = nst > 0 ? nst - 1 : 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) gload(bufs[b], r0 + (int64_t)(b < last ? b : last) * SR);
    if (nst > 0) lstore(bufs[0], 0, r0);
    gload(bufs[0], r0 + (int64_t)(NB < last ? NB : last) * SR);
    lds_sync();
    for (int st = 0; st < nst; st += NB) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int sc = st + u;                     // stage in LDS[sc & 1]
        if (sc >= nst) break;
        compute(sc & 1, r0 + (int64_t)sc * SR);
        __builtin_amdgcn_sched_barrier(0);
        if (sc + 1 < nst) lstore(bufs[(u + 1) % NB], (sc + 1) & 1, r0 + (int64_t)(sc + 1) * SR);
        gload(bufs[(u + 1) % NB], r0 + (int64_t)(sc + 1 + NB < last ? sc + 1 + NB : last) * SR);
        lds_sync();
      }
    }
  } else {
    // large tiles (one wave per SIMD): one register buffer, one stage ahead
    uint4 b0[PPT][RPP];
    if (nst > 0) {
      gload(b0, r0);
      lstore(b0, 0, r0);
    }
    lds_sync();
    for (int st = 0; st < nst; ++st) {
      gload(b0, r0 + (int64_t)(st + 1 < nst ? st + 1 : st) * SR);
      compute(st & 1, r0 + (int64_t)st * SR);
      __builtin_amdgcn_sched_barrier(0);
      if (st + 1 < nst) lstore(b0, (st + 1) & 1, r0 + (int64_t)(st + 1) * SR);
      lds_sync();
    }
  }

  const int hh = lane >> 5;
  const int64_t obase = ((int64_t)g * n_split + split) * (int64_t)N * J;
  if constexpr (PM == PM_F64) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int j = j0 + 32 * wn + 16 * b + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int n = n0 + 32 * wm + 16 * a + (lane >> 4) + 4 * r;
          if (n < N && j < J) partial64[obase + (int64_t)n * J + j] = accd[a][b][r];
        }
      }
  }
#pragma unroll
  for (int a = 0; a < (PM == PM_F64 ? 0 : NT); ++a) {
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      const int j = j0 + 32 * (wn * NT + b) + (lane & 31);
      if (j >= J) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int n = n0 + 32 * (wm * NT + a) + 8 * (r >> 2) + 4 * hh + (r & 3);
        if (n >= N) continue;
        partial[obase + (int64_t)n * J + j] = acc[a][b][r];
      }
    }
  }
  if (pdb && tj == 0 && tid < BNn && n0 + tid < N)
    pdb[((int64_t)g * n_split + split) * N + n0 + tid] = dbacc;
}

// ---------------------------------------------------------------------------
// k_gemm_dw_tr: the same weight gradient for 16-bit storage, with row-major
// operand stages in LDS.  Global loads are whole 16-byte row segments, 16
// lanes per 256-byte row (fully used cache lines); the matrix-core fragments,
// which need 8 consecutive rows of one column per lane, are gathered with the
// transposing LDS read of gfx950: within each 16-lane group, lanes 4r..4r+3
// address the four 8-byte pieces of row r of a 4 x 16 block and lane i
// receives column i of the block.  Two such reads give a lane its 8 rows.
// Row pitch = row bytes + pad with pitch/4 = 16 or 48 (mod 64), so the four
// rows of one read fall in disjoint bank ranges.
// ---------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 tr_bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(__fp16)))) __fp16 tr_f16x4;

template <class T>
__device__ __forceinline__ u32x2 lds_read_tr(const char* p) {
  if constexpr (__is_same(T, bf16)) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                                         (__attribute__((address_space(3))) tr_bf16x4*)(p)));
  } else {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4f16(
                                         (__attribute__((address_space(3))) tr_f16x4*)(p)));
  }
}

// The same transposing read issued as an instruction the compiler does not
// model.  Stages filled by LDS DMA (global_load_lds) are guarded by explicit
// vmcnt waits and barriers; with the intrinsic, the compiler cannot tell the
// DMA targets apart from the stage being read and drains every DMA in flight
// (vmcnt(0)) before each stage's reads, which leaves nothing prefetched.  The
// caller waits for these reads itself (lgkm_wait below).
__device__ __forceinline__ u32x2 lds_read_tr_raw(const char* p) {
  const uint32_t a = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
  u32x2 r;
  asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(r) : "v"(a));
  return r;
}

// s_waitcnt lgkmcnt(N) that the values read before it flow through, so no
// use of them is scheduled ahead of the wait
template <int N, int K>
__device__ __forceinline__ void lgkm_wait(u32x4 (&v)[K]) {
  static_assert(N >= 0 && N <= 15, "lgkmcnt range");
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
#pragma unroll
  for (int i = 0; i < K; ++i) asm volatile("" : "+v"(v[i]));
}

__host__ __device__ constexpr int dw_tr_pitch(int row_bytes) {
  // smallest pitch >= row_bytes (multiple of 64 bytes) with pitch/4 = 16 or 48 mod 64
  return (row_bytes / 4) % 64 == 16 || (row_bytes / 4) % 64 == 48 ? row_bytes
         : (row_bytes / 4) % 64 == 0 ? row_bytes + 64 : row_bytes + 64 * ((row_bytes / 4) % 64 == 32 ? 1 : 0);
}

// NS > 0 (tile sides of 128 or 256 columns): the stages move straight from
// global memory into an NS-deep LDS ring (global_load_lds_dwordx4).  Rows are
// then unpadded (256 or 512 bytes); the 16-byte segment s of row r sits at
// s ^ 4 (r & 3), which keeps the four rows of a transposing read in disjoint
// bank ranges.
template <class T, int WM, int WN, int NT, int NB, int NS = 0, int OCC = 2>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC)))
k_gemm_dw_tr(const T* __restrict__ dA, int64_t a_g, int64_t lda, const T* __restrict__ H, int64_t h_g,
             int64_t ldh, int64_t R, int64_t n_value, int N, int J, float* __restrict__ partial,
             double* __restrict__ pdb, int n_split, int64_t rows_per_split) {
  static_assert(sizeof(T) == 2, "16-bit storage only");
  constexpr int BNn = 32 * NT * WM;
  constexpr int BJ = 32 * NT * WN;
  constexpr int NTH = 64 * WM * WN;
  constexpr int SR = 32;                    // rows per stage (two 16-row k chunks)
  constexpr int SA = BNn / 8, SB = BJ / 8;  // 16-byte segments per row
  constexpr int PA = dw_tr_pitch(BNn * 2), PB = dw_tr_pitch(BJ * 2);
  constexpr int REGA = SR * PA;
  constexpr int STAGE = REGA + SR * PB;
  constexpr int PIECES = SR * (SA + SB);
  static_assert(PIECES % NTH == 0, "whole pieces per thread");
  constexpr int PPT = PIECES / NTH;
  static_assert(NS == 0 || ((BNn == 128 || BNn == 256) && (BJ == 128 || BJ == 256) && NS >= 2),
                "direct-to-LDS stages: tile sides of 128 or 256");
  constexpr int RBA = BNn * 2, RBB = BJ * 2;  // unpadded ring row bytes
  constexpr int DSTAGE = SR * (RBA + RBB);    // ring stage: SR rows of A, then SR rows of B
  constexpr int LDSB = NS > 0 ? NS * DSTAGE : 2 * STAGE;
  typedef typename Elem<T>::frag frag;
  __shared__ __attribute__((aligned(16))) char lds[LDSB];

  const int tiles_n = (N + BNn - 1) / BNn;
  const int tiles = tiles_n * ((J + BJ - 1) / BJ);
  const int64_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = (int)(lb % tiles);
  const int tn = tile % tiles_n;
  const int tj = tile / tiles_n;
  const int split = (int)(lb / tiles);
  const int g = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % WM;
  const int wn = wave / WM;
  const int n0 = tn * BNn;
  const int j0 = tj * BJ;
  // stages are dealt round-robin over the splits (split s takes stages s,
  // s + n_split, ...), so at any time the blocks stream one contiguous window
  // of rows (page and DRAM locality) instead of n_split separate ranges
  (void)rows_per_split;
  const int64_t r1 = R;
  const int64_t rv = R < n_value ? R : n_value;
  const int64_t tot = (R + SR - 1) / SR;
  const int nst = (int)(split < tot ? (tot - split + n_split - 1) / n_split : 0);
  auto krow = [&](int sc) { return ((int64_t)split + (int64_t)sc * n_split) * SR; };
  const T* A = dA + g * a_g;
  const T* B = H + g * h_g;

  f32x16 acc[NT][NT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
  float dbp[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) dbp[t] = 0.0f;
  double dbacc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) dbacc[t] = 0.0;
  const bool want_db = pdb && tj == 0 && wn == 0;

  // piece q: operand A for q < SR * SA (row q / SA, segment q % SA), else B.
  // Rows past the range load a clamped row and are zeroed at the LDS store;
  // columns past the end load a clamped column (never stored outputs).
  auto gload = [&](u32x4* buf, int64_t k0) {
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int q = tid + i * NTH;
      const bool isA = q < SR * SA;
      const int qq = isA ? q : q - SR * SA;
      const int sg = isA ? qq % SA : qq % SB;
      const int row = isA ? qq / SA : qq / SB;
      int64_t gr = k0 + row;
      if (gr >= r1) gr = r1 - 1;
      int col = (isA ? n0 : j0) + sg * 8;
      const int lim = isA ? N : J;
      if (col >= lim) col = lim - 8;
      buf[i] = isA ? *(const u32x4*)(A + gr * lda + col) : *(const u32x4*)(B + gr * ldh + col);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto lstore = [&](const u32x4* buf, int stage, int64_t k0) {
    char* base = lds + stage * STAGE;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int q = tid + i * NTH;
      const bool isA = q < SR * SA;
      const int qq = isA ? q : q - SR * SA;
      const int sg = isA ? qq % SA : qq % SB;
      const int row = isA ? qq / SA : qq / SB;
      const uint32_t m = (k0 + row < r1) ? 0xffffffffu : 0u;
      const u32x4 v = buf[i] & m;
      *(u32x4*)(base + (isA ? row * PA : REGA + row * PB) + sg * 16) = v;
    }
  };
  // fragments: lane l holds rows 8 (l / 32) .. +7 of its column (l % 32) of
  // the 32-column block, as two transposing reads of 4 rows
  const int grp = lane >> 4, t16 = lane & 15;
  const int rr = t16 >> 2, qq4 = t16 & 3;
  const int kb = 8 * (lane >> 5);
  auto frag_at = [&](const char* region, int pitch, int c, int colblk) {
    const int byte = (colblk + 16 * (grp & 1) + 4 * qq4) * 2;
    // the row of both reads is = rr (mod 4): one swizzle for the pair
    const char* p0 = NS > 0 ? region + (c * 16 + kb + rr) * pitch + (((byte >> 4) ^ (4 * rr)) << 4) + (byte & 15)
                            : region + (c * 16 + kb + rr) * pitch + byte;
    const u32x2 lo = lds_read_tr<T>(p0);
    const u32x2 hi = lds_read_tr<T>(p0 + 4 * pitch);
    const u32x4 w = {lo.x, lo.y, hi.x, hi.y};
    return __builtin_bit_cast(frag, w);
  };
  // DMA stages: raw transposing reads of the fragments.  Four-wave blocks
  // read both 16-row chunks up front and start the first chunk's products
  // once its reads have landed; larger blocks (which would lose occupancy to
  // the extra registers) read one chunk at a time.
  auto frag_raw = [&](const char* region, int pitch, int c, int colblk) {
    const int byte = (colblk + 16 * (grp & 1) + 4 * qq4) * 2;
    const char* p0 = region + (c * 16 + kb + rr) * pitch + (((byte >> 4) ^ (4 * rr)) << 4) + (byte & 15);
    const u32x2 lo = lds_read_tr_raw(p0);
    const u32x2 hi = lds_read_tr_raw(p0 + 4 * pitch);
    return u32x4{lo.x, lo.y, hi.x, hi.y};
  };
  auto compute_dma = [&](int stage, int64_t k0) {
    static_assert(SR == 32, "two 16-row chunks per stage");
    const char* base = lds + stage * DSTAGE;
    const char* bbase = base + SR * RBA;
    constexpr bool AHEAD = NTH <= 256;
    u32x4 w[2][2 * NT];   // chunk c: A fragments 0..NT-1, then B fragments
    auto read_chunk = [&](int c) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        w[c][t] = frag_raw(base, RBA, c, 32 * (wm * NT + t));
        w[c][NT + t] = frag_raw(bbase, RBB, c, 32 * (wn * NT + t));
      }
    };
    read_chunk(0);
    if constexpr (AHEAD) read_chunk(1);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (c == 1 && !AHEAD) read_chunk(1);
      if (c == 0 && AHEAD) lgkm_wait<4 * NT>(w[0]);   // the second chunk's 4 NT reads may still be in flight
      else lgkm_wait<0>(w[c]);
      frag af[NT], bf[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        af[t] = __builtin_bit_cast(frag, w[c][t]);
        bf[t] = __builtin_bit_cast(frag, w[c][NT + t]);
      }
      // the stages hold clamped copies of the last row past R: their dA
      // elements (rows k0 + 16 c + kb + e of this lane) contribute zero
      if (k0 + SR > r1) {
        const int64_t rw0 = k0 + c * 16 + kb;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (rw0 + e >= r1) af[t][e] = Elem<T>::from_f(0.0f);
      }
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) Elem<T>::mma(acc[a][b], af[a], bf[b]);
      if (want_db && k0 + c * 16 < rv) {
        const int64_t rw0 = k0 + c * 16 + kb;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e) dbp[t] += rw0 + e < rv ? Elem<T>::to_f(af[t][e]) : 0.0f;
      }
    }
    if (want_db) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        dbacc[t] += (double)dbp[t];
        dbp[t] = 0.0f;
      }
    }
  };
  auto compute = [&](int stage, int64_t k0) {
    const char* base = lds + stage * (NS > 0 ? DSTAGE : STAGE);
    const char* bbase = base + (NS > 0 ? SR * RBA : REGA);
#pragma unroll
    for (int c = 0; c < SR / 16; ++c) {
      frag af[NT], bf[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        af[t] = frag_at(base, NS > 0 ? RBA : PA, c, 32 * (wm * NT + t));
        bf[t] = frag_at(bbase, NS > 0 ? RBB : PB, c, 32 * (wn * NT + t));
      }
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) Elem<T>::mma(acc[a][b], af[a], bf[b]);
      // bias cotangent: value rows of the lane's 8 rows of its dA columns
      if (want_db && k0 + c * 16 < rv) {
        const int64_t rw0 = k0 + c * 16 + kb;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e) dbp[t] += rw0 + e < rv ? Elem<T>::to_f(af[t][e]) : 0.0f;
      }
    }
    if (want_db) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        dbacc[t] += (double)dbp[t];
        dbp[t] = 0.0f;
      }
    }
  };

  if constexpr (NS > 0) {
    // One DMA instruction of a wave fills 1 KB: 1024 / RB rows of one
    // operand (RB = its row bytes), lane l at byte 16 l (physical segment
    // l % (RB / 16) of its row, holding the logical segment of that index
    // ^ 4 (row & 3)).  A stage is GA such groups of A rows and GB of B rows,
    // dealt to the waves round-robin.  Rows past R (in the last stage, at
    // most) load a clamped row; compute() zeroes their dA elements.  Every
    // stage is a DMA stage, so the waits below are the only ones on the
    // ring (a register-loaded stage made the compiler drain every load in
    // flight before each stage's LDS reads).
    constexpr int GA = SR * RBA / 1024, GB = SR * RBB / 1024;
    constexpr int NG = GA + GB;
    constexpr int NW = NTH / 64;
    static_assert(NG % NW == 0, "whole row groups per wave");
    constexpr int GPW = NG / NW;
    static_assert((NS - 2) * GPW <= 63, "outstanding loads exceed the vmcnt range");
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T* dsrc[GPW];
    int64_t dld[GPW];
    int drow[GPW];
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
      const int gq = wv + i * NW;
      const bool isA = gq < GA;
      const int spr = (isA ? RBA : RBB) / 16;  // segments per row
      const int row = (isA ? gq : gq - GA) * (64 / spr) + lane / spr;
      const int sg = (lane % spr) ^ (4 * (row & 3));
      int col = (isA ? n0 : j0) + sg * 8;
      const int lim = isA ? N : J;
      if (col >= lim) col = lim - 8;
      dsrc[i] = (isA ? A : B) + col;
      dld[i] = isA ? lda : ldh;
      drow[i] = row;
    }
    auto issue = [&](int sc, int buf) {
      const int64_t k0 = krow(sc);
      char* dst = lds + buf * DSTAGE;
#pragma unroll
      for (int i = 0; i < GPW; ++i) {
        int64_t gr = k0 + drow[i];
        if (gr > r1 - 1) gr = r1 - 1;
        __builtin_amdgcn_global_load_lds((const void*)(dsrc[i] + gr * dld[i]),
                                         (lds_ptr_t)(dst + (wv + i * NW) * 1024), 16, 0, 0);
      }
    };
#pragma unroll
    for (int b = 0; b < NS - 1; ++b)
      if (b < nst) issue(b, b);
    int stg = 0;
    for (int sc = 0; sc < nst; ++sc) {
      const int later = nst - 1 - sc;
      if constexpr (NS >= 4) {
        if (later >= 2) wait_vmcnt<2 * GPW>();
        else if (later == 1) wait_vmcnt<GPW>();
        else wait_vmcnt<0>();
      } else if constexpr (NS == 3) {
        if (later >= 1) wait_vmcnt<GPW>();
        else wait_vmcnt<0>();
      } else {
        wait_vmcnt<0>();
      }
      lds_sync();
      if (sc + NS - 1 < nst) issue(sc + NS - 1, stg == 0 ? NS - 1 : stg - 1);
      compute_dma(stg, krow(sc));
      stg = stg + 1 == NS ? 0 : stg + 1;
    }
  } else {
  // ring of NB register stages (as in k_gemm_dw)
  u32x4 bufs[NB][PPT];
  const int last = nst > 0 ? nst - 1 : 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) gload(bufs[b], krow(b < last ? b : last));
  if (nst > 0) lstore(bufs[0], 0, krow(0));
  gload(bufs[0], krow(NB < last ? NB : last));
  lds_sync();
  for (int st = 0; st < nst; st += NB) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int sc = st + u;
      if (sc >= nst) break;
      compute(sc & 1, krow(sc));
      __builtin_amdgcn_sched_barrier(0);
      if (sc + 1 < nst) lstore(bufs[(u + 1) % NB], (sc + 1) & 1, krow(sc + 1));
      gload(bufs[(u + 1) % NB], krow(sc + 1 + NB < last ? sc + 1 + NB : last));
      lds_sync();
    }
  }
  }

  const int hh = lane >> 5;
  float* out = partial + ((int64_t)g * n_split + split) * (int64_t)N * J;
#pragma unroll
  for (int a = 0; a < NT; ++a) {
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      const int j = j0 + 32 * (wn * NT + b) + (lane & 31);
      if (j >= J) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int n = n0 + 32 * (wm * NT + a) + 8 * (r >> 2) + 4 * hh + (r & 3);
        if (n < N) out[(int64_t)n * J + j] = acc[a][b][r];
      }
    }
  }
  if (want_db) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      double v = dbacc[t];
      v += __shfl_xor(v, 32);                      // the other 8-row half of the same column
      const int n = n0 + 32 * (wm * NT + t) + (lane & 31);
      if (lane < 32 && n < N) pdb[((int64_t)g * n_split + split) * N + n] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// Tiles.  A wave owns 32 points x 32*NT columns of every stream.  16-bit
// forwards (two-term weights) and reverse passes of 128 columns and more whose
// contraction is whole 128-byte slices take the ring kernels (ring_ok), 128 x
// 128 layers of up to five streams the resident kernel; fp32-stored products of
// one and two streams with few output tiles the short kernels.  The others are
// register-staged: NT = 4 / 2 / 1 for 1 / 2 / 3+ streams (2 x 2 waves, two waves
// per SIMD), and 4 x 1 waves for narrow layers (N <= 32).

bool nt_resident_ok(int elem_bytes, int C, int K, int N, int64_t n_points, int64_t ldx, int64_t ldo) {
  const int64_t span = (n_points + 1) * (ldx > ldo ? ldx : ldo) * (int64_t)elem_bytes;
  return elem_bytes == 2 && C >= 1 && C <= 5 && K == 128 && N == 128 && span < ((int64_t)1 << 31);
}

// The fused launch saves one write and one read of every top activation, but
// runs on the 32 x 128 tile: on the large ones the column weights push the
// accumulators out of the register file (five streams at K = 512 1917 us, three
// 1854).  us per launch, fused | the faster tile and a separate pass, 262,144
// points at K = N = 256 and 512, 131,072 at 768 and 1024, 32,768 at 2048:
//            K = 256     512           768           1024          2048
//   C = 3    407 | 502   1225 | 1200   1208 | 1135   2055 | 1813   1935 | 1596
//   C = 4    461 | 646   1338 | 1771   1440 | 1775   2280 | 2818   2201 | 2589
//   C = 5    575 | 805   1725 | 2040   1736 | 1989   2882 | 3059   2807 | 2724
//   C = 7    964 | 1110  2963 | 2980   3205 | 3076   5124 | 4694   4743 | 4162
// (Five streams at 1024 and 262,144 points: 6.02 | 5.96 ms, the 6 x 1024 step
// 1783 | 1778 ms.)  One and two streams stay on the large tiles (value fields of
// width 512, 8.34 ms fused, 7.17 apart).
bool nt_ring_out_ok(int elem_bytes, int C, int K, int N, int64_t n_points) {
  const bool pays = C == 4 || (C == 5 && N <= 768) || ((C == 3 || C == 7) && N <= 256);
  return elem_bytes == 2 && pays && K == N && N >= 128 && N % 128 == 0 && n_points > 0 &&
         !nt_resident_ok(elem_bytes, C, K, N, n_points, K, N);
}

namespace {

// compute units of the current device (cached per device)
int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (cached[dev] <= 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// launches of the ring kernels: whole 128-byte k slices, and the arrays' rows
// addressable from a tile's first row with 32-bit offsets (a tile spans at
// most 256 rows)
template <class T, int C, int EPI>
bool ring_ok(const NtArgs<T>& a) {
  const int kx = a.kx > 0 ? a.kx : a.K;
  return sizeof(T) == 2 && (EPI == EPI_FWD) == (a.kx > 0) && a.N >= 128 &&
         kx >= 128 && kx % 64 == 0 && a.ldx < (1 << 22) && a.ldw < (1 << 22);
}

template <class T, int ND1, int ND2, int EPI>
hipError_t nt_dispatch_tile(const NtArgs<T>& a, int G, hipStream_t st) {
  constexpr int C = 1 + ND1 + ND2;
  constexpr int NTM = C == 1 ? 4 : (C == 2 ? 2 : 1);
  const int64_t npts = a.seg.n_points;
  if (npts <= 0) return hipSuccess;
  if (EPI == EPI_FWD && !a.bias) return hipErrorInvalidValue;
  if ((a.pm != PM_NATIVE && a.pm != PM_SPLIT2 && a.pm != PM_F64) || (a.pm != PM_NATIVE && sizeof(T) != 4) ||
       (a.kx > 0 && (sizeof(T) != 2 || a.K != 2 * a.kx)))
    return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 4) {
    // split products (the critic and the generators' sensor rows): one or two
    // streams; register-staged tiles
    if (a.pm != PM_NATIVE) {
      // (nor one row per stream: the short kernels read whole ones)
      if (a.y || a.fp1 || a.a_seeds) return hipErrorInvalidValue;
      if constexpr (C <= 2) {
        // few output tiles.  us per forward launch, tiled -> short, rows x N x K
        // (number of 32 x 32 blocks): split products 512 x 256 x 416 (128)
        // 28.0 -> 10.1, 192 x 2048 x 8192 (384) 374 -> 122, 1024 x 1024 x 1024
        // (1024) 58.6 -> 39.1, 4096 x 256 x 256 (1024) 22.0 -> 17.2 but 2048
        // blocks 23.6 -> 29.3; K = 128: 512 blocks 12.1 -> 9.4, 1024 12.8 ->
        // 13.9.  fp64 products 512 x 256 x 416 26.6 -> 10.6, 4096 x 128 x 128
        // (512) 14.2 -> 10.5, 1024 blocks 15.2 -> 15.5
        const int64_t sblocks = ((npts + 31) / 32) * (a.N / 32) * G;
        const int64_t limit = (a.pm == PM_F64 ? 3 : a.K >= 256 ? 4 : 2) * (int64_t)cu_count();
        if (a.N % 32 == 0 && a.K % 16 == 0 && sblocks <= limit) {
          dim3 grid((unsigned)(((npts + 31) / 32) * (a.N / 32)), 1, G);
          if (a.pm == PM_SPLIT2) k_gemm_short_x2<ND1, EPI><<<grid, 64, 0, st>>>(a);
          else if (a.K >= 1024) k_gemm_short<ND1, EPI, 8><<<grid, 512, 0, st>>>(a);   // (eight waves share the contraction)
          else k_gemm_short<ND1, EPI, 4><<<grid, 256, 0, st>>>(a);
          return hipGetLastError();
        }
        if (a.N <= 32 && a.pm != PM_F64) {
          dim3 grid((unsigned)(((npts + 127) / 128) * ((a.N + 31) / 32)), 1, G);
          k_gemm_nt<T, ND1, ND2, 4, 1, 1, 1, EPI, 2, true, false, PM_SPLIT2><<<grid, 256, 0, st>>>(a);
        } else if (a.pm == PM_SPLIT2 && C == 1 && a.N >= 256 && npts * G >= 16384 && a.K % 32 == 0) {
          // sensor rows: 128 points x 256 columns, stages of two k slices (a
          // whole 128-byte line of every row at once).  us per forward launch
          // at K = N, 262,144 rows (one slice per stage -> two): 1024 1930 ->
          // 1829 (reverse 1849 -> 1743), 512 592 -> 593 (577 -> 557); at 256
          // eight waves of 2 x 2 fragments, 229 -> 213 (16 waves of 1 x 2 215
          // -> 208 in the reverse)
          if constexpr (C == 1) {
            dim3 grid((unsigned)(((npts + 127) / 128) * ((a.N + 255) / 256)), 1, G);
            if (a.K >= 512) k_gemm_nt<T, ND1, ND2, 4, 4, 1, 2, EPI, 1, true, false, PM_SPLIT2, 3, 2><<<grid, 1024, 0, st>>>(a);
            else if (EPI == EPI_FWD) k_gemm_nt<T, ND1, ND2, 2, 4, 2, 2, EPI, 1, true, false, PM_SPLIT2, 2, 2><<<grid, 512, 0, st>>>(a);
            else k_gemm_nt<T, ND1, ND2, 4, 4, 1, 2, EPI, 1, true, false, PM_SPLIT2, 2, 2><<<grid, 1024, 0, st>>>(a);
          }
        } else if (a.pm == PM_SPLIT2 && C == 1 && a.N <= 128) {
          // no idle column half at N = 128: 64 points x 128 columns, 2 x 2
          // waves; 128 points and whole-line stages where the arrays outgrow
          // the memory-side cache (us per launch at K = 128, 131,072 rows:
          // 42.0 against 45.1, reverse 40.2 against 40.4; 262,144 rows: 122
          // against 110, reverse 108 against 99)
          if constexpr (C == 1) {
            if constexpr (EPI != EPI_DF) {
              if (a.N == 128 && npts * G >= 196608 && a.K % 32 == 0) {
                dim3 grid((unsigned)((npts + 127) / 128), 1, G);
                k_gemm_nt<T, ND1, ND2, 2, 2, 2, 2, EPI, 2, true, false, PM_SPLIT2, 2, 2><<<grid, 256, 0, st>>>(a);
                return hipGetLastError();
              }
            }
            dim3 grid((unsigned)(((npts + 63) / 64) * ((a.N + 127) / 128)), 1, G);
            k_gemm_nt<T, ND1, ND2, 2, 2, 1, 2, EPI, 2, true, false, PM_SPLIT2><<<grid, 256, 0, st>>>(a);
          }
        } else if (a.pm == PM_SPLIT2) {
          // 64 points x 64 NTM columns, 2 x 2 waves
          constexpr int BN = 64 * NTM;
          dim3 grid((unsigned)(((npts + 63) / 64) * ((a.N + BN - 1) / BN)), 1, G);
          k_gemm_nt<T, ND1, ND2, 2, 2, 1, NTM, EPI, 2, true, false, PM_SPLIT2><<<grid, 256, 0, st>>>(a);
        } else {
          // fp64 products: 64 x 64 tiles
          dim3 grid((unsigned)(((npts + 63) / 64) * ((a.N + 63) / 64)), 1, G);
          k_gemm_nt<T, ND1, ND2, 2, 2, 1, 1, EPI, 2, true, false, PM_F64><<<grid, 256, 0, st>>>(a);
        }
        return hipGetLastError();
      } else {
        return hipErrorInvalidValue;
      }
    }
  }
  if constexpr (sizeof(T) == 2 && C <= 5) {
    const bool skip = a.skip || a.skip_g || a.out_gh;
    const bool two = a.kx > 0;   // two-term weight rows: the operand is kx wide
    if (nt_resident_ok((int)sizeof(T), C, two ? a.kx : a.K, a.N, npts, a.ldx, a.ldo) &&
        !(skip && (a.fp1 || a.y)) && (!two || (EPI == EPI_FWD && a.K == 2 * a.kx))) {
      // persistent weight-resident kernel: two blocks per CU in total (one
      // for the five-stream skip variant)
      const int64_t ntiles = (npts + 31) / 32;
      // one-stream launches (sensor rows: few tiles, small blocks) take three
      // blocks per CU
      int64_t nb = (skip || (two && C >= 5) ? wr_blocks_per_cu<C, true>() : (C == 1 ? 3 : 2)) * (int64_t)cu_count() / G;
      if (nb < 1) nb = 1;
      if (nb > ntiles) nb = ntiles;
      dim3 grid((unsigned)nb, 1, G);
      if constexpr (EPI == EPI_FWD) {
        if (two) {
          if (a.fp1) k_gemm_nt_wr<T, ND1, ND2, EPI, true, false, true><<<grid, 256, 0, st>>>(a, ntiles);
          else if (skip) k_gemm_nt_wr<T, ND1, ND2, EPI, false, true, true><<<grid, 256, 0, st>>>(a, ntiles);
          else k_gemm_nt_wr<T, ND1, ND2, EPI, false, false, true><<<grid, 256, 0, st>>>(a, ntiles);
          return hipGetLastError();
        }
      }
      if (a.a_seeds && !a.fp1 && !skip) return hipErrorInvalidValue;
      if (a.fp1) k_gemm_nt_wr<T, ND1, ND2, EPI, true><<<grid, 256, 0, st>>>(a, ntiles);
      else if (skip) k_gemm_nt_wr<T, ND1, ND2, EPI, false, true><<<grid, 256, 0, st>>>(a, ntiles);
      else k_gemm_nt_wr<T, ND1, ND2, EPI, false><<<grid, 256, 0, st>>>(a, ntiles);
      return hipGetLastError();
    }
  }
  // the first layer is fused only in the resident kernel, the output layer in
  // the ring kernels too
  if (a.fp1 || (a.y && !(C >= 3 && !a.skip && ring_ok<T, C, EPI>(a) && a.ypart && a.N % 128 == 0))) return hipErrorInvalidValue;
  if constexpr (EPI == EPI_DF) {
    if (a.skip || a.skip_g || a.out_gh) return hipErrorInvalidValue;
  }
  if (a.N <= 32) {
    dim3 grid((unsigned)(((npts + 127) / 128) * ((a.N + 31) / 32)), 1, G);
    k_gemm_nt<T, ND1, ND2, 4, 1, 1, 1, EPI, (C >= 4 ? 1 : 2)><<<grid, 256, 0, st>>>(a);
  } else if (ring_ok<T, C, EPI>(a)) {
    // 16-bit layers of 128 columns and more (128 itself: what the resident
    // kernel does not take): operand stages straight into LDS.  Large tiles
    // (eight waves) read every operand fewer times and suit the
    // matrix-core-bound depths; 32 points x 128 columns (four waves, two blocks
    // per CU for up to five streams, so that one block's epilogue runs beside
    // the other's products) suits launches that would give the chip fewer than
    // two rounds of large tiles, and where the figures say so.  us per launch,
    // large | 32 x 128, points as in nt_ring_out_ok's table:
    //                K = N = 256   512           768           1024          2048
    //   forward C=1    528 | 725   1378 | 2126   1311 | 2191   2198 | 4175   1960 | 8610   (4 x the points)
    //           C=2    300 | 334   725 | 909     687 | 947     1112 | 1595   968 | 1597
    //           C=3    405 | 452   1010 | 1370   982 | 1341    1630 | 2149   1472 | 2039
    //           C=4    575 | 521   1700 | 1548   1715 | 1606   2836 | 2601   2570 | 2439
    //           C=5    700 | 670   1730 | 1922   1732 | 1951   2757 | 3119   2513 | 2954
    //           C=7    900 | 1062  2590 | 3114   2780 | 3348   4312 | 5404   3905 | 4889
    //   reverse C=2    235 | 214   580 | 556     535 | 546     831 | 879     685 | 837
    //           C=3    308 | 310   751 | 877     700 | 842     1087 | 1317   907 | 1153
    //           C=4    432 | 374   1193 | 1030   1100 | 940    1800 | 1514   1540 | 1321
    //           C=5    568 | 480   1446 | 1217                 2022 | 1869
    // (seven streams reverse: 32 x 128 only)
    if constexpr (sizeof(T) == 2) {
      constexpr bool FWD = EPI == EPI_FWD;
      constexpr int WM = C == 1 ? 4 : 2, WN = C == 1 ? 2 : 4, MT = C <= 3 && FWD ? 2 : 1, NT = C == 1 ? 4 : (C <= 3 || C == 5 ? 2 : 1);
      constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN;
      const int64_t blocks = ((npts + BM - 1) / BM) * ((a.N + BN - 1) / BN) * G;
      constexpr int LARGE_N = FWD ? (C == 5 ? 512 : 256) : (C == 2 ? 768 : 512);   // narrowest that takes the large tile
      const bool large = !a.y && a.N >= LARGE_N && blocks >= 2 * (int64_t)cu_count();
      if constexpr (C != 4 && (FWD || C <= 3)) {
        if (large) {
          dim3 grid((unsigned)(((npts + BM - 1) / BM) * ((a.N + BN - 1) / BN)), 1, G);
          k_gemm_nt<T, ND1, ND2, WM, WN, MT, NT, EPI, 1, true, true, PM_NATIVE, 2><<<grid, 64 * WM * WN, 0, st>>>(a);
          return hipGetLastError();
        }
      }
      dim3 grid((unsigned)(((npts + 31) / 32) * ((a.N + 127) / 128)), 1, G);
      if constexpr (FWD && C >= 3) {
        if (a.y) {
          k_gemm_nt<T, ND1, ND2, 1, 4, 1, 1, EPI, (C <= 5 ? 2 : 1), true, true, PM_NATIVE, 2, 1, true><<<grid, 256, 0, st>>>(a);
          if (a.N > 128)
            k_out_sum<<<dim3((unsigned)((C * npts + 255) / 256), 1, G), 256, 0, st>>>(
                a.ypart, a.yp_g, a.N / 128, npts, C, a.seg, a.wout, a.wo_g, a.N, a.y, a.y_g);
          return hipGetLastError();
        }
      }
      k_gemm_nt<T, ND1, ND2, 1, 4, 1, 1, EPI, (C <= 5 ? 2 : 1), true, true, PM_NATIVE, 2><<<grid, 256, 0, st>>>(a);
    } else {
      return hipErrorInvalidValue;
    }
  } else {
    constexpr int BN = 64 * NTM;
    dim3 grid((unsigned)(((npts + 63) / 64) * ((a.N + BN - 1) / BN)), 1, G);
    k_gemm_nt<T, ND1, ND2, 2, 2, 1, NTM, EPI, (C >= 7 ? 1 : 2)><<<grid, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

template <class T, int EPI>
hipError_t nt_dispatch_streams(int nd1, int nd2, const NtArgs<T>& a, int G, hipStream_t st) {
  const int key = nd1 * 10 + nd2;
  // (one stream backward is the sensor rows' and the critic's, whose storage is fp32)
  if constexpr (sizeof(T) == 2 && EPI == EPI_BWD) {
    if (key == 0) return hipErrorInvalidValue;
  } else {
    if (key == 0) return nt_dispatch_tile<T, 0, 0, EPI>(a, G, st);
  }
  switch (key) {
    case 10: return nt_dispatch_tile<T, 1, 0, EPI>(a, G, st);
    case 20: return nt_dispatch_tile<T, 2, 0, EPI>(a, G, st);
    case 30: return nt_dispatch_tile<T, 3, 0, EPI>(a, G, st);
    case 11: return nt_dispatch_tile<T, 1, 1, EPI>(a, G, st);
    case 22: return nt_dispatch_tile<T, 2, 2, EPI>(a, G, st);
    case 33: return nt_dispatch_tile<T, 3, 3, EPI>(a, G, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

template <class T>
hipError_t launch_gemm_nt(int epi, int nd1, int nd2, const NtArgs<T>& a, int G, hipStream_t st) {
  if (epi == EPI_FWD) return nt_dispatch_streams<T, EPI_FWD>(nd1, nd2, a, G, st);
  if (epi == EPI_BWD) return nt_dispatch_streams<T, EPI_BWD>(nd1, nd2, a, G, st);
  if constexpr (sizeof(T) == 4) {   // (the critic's storage)
    if (nd1 == 0 && nd2 == 0) return nt_dispatch_tile<T, 0, 0, EPI_DF>(a, G, st);
  }
  return hipErrorInvalidValue;
}

void dw_split_plan(int64_t R, int N, int J, int elem_bytes, int G, int* n_split, int64_t* rows_per_split) {
  const int SR = 64 / elem_bytes;
  // 16-bit storage, both sides >= 512: 256 x 256 tiles of 16 waves, about
  // 256 blocks (one per CU; as fast as 512 and half the partials to write and
  // reduce); otherwise about 1024 blocks of the 128 x 128 (or smaller) tile
  // grid, and 512 for a single output tile (each split writes a whole N x J
  // fp32 partial, and one resident wave of blocks suffices)
  const bool big = elem_bytes == 2 && N >= 512 && J >= 512;
  const int bt = big ? 256 : (N >= 128 && J >= 128) ? 128 : ((N >= 64 && J >= 64) ? 64 : 32);
  const int64_t tiles = (int64_t)((N + bt - 1) / bt) * ((J + bt - 1) / bt) * G;
  const int64_t target = big ? 256 : (tiles == 1 ? 512 : 1024);
  int64_t want = (target + tiles - 1) / tiles;
  const int64_t stages = (R + SR - 1) / SR;
  int64_t max_split = stages / 4 > 0 ? stages / 4 : 1;
  if (want > max_split) want = max_split;
  if (want < 1) want = 1;
  if (want > 65535) want = 65535;
  int64_t rps = (R + want - 1) / want;
  rps = (rps + SR - 1) / SR * SR;
  if (rps <= 0) rps = SR;
  *rows_per_split = rps;
  *n_split = (int)((R + rps - 1) / rps);
  if (*n_split < 1) *n_split = 1;
}

template <class T>
hipError_t launch_gemm_dw(const T* dA, int64_t a_g, int64_t lda, const T* H, int64_t h_g, int64_t ldh,
                          int64_t R, int64_t n_value, int N, int J, float* partial, double* pdb,
                          int n_split, int64_t rows_per_split, int G, hipStream_t st, int pm, double* partial64) {
  if (R <= 0) return hipSuccess;
  if ((pm != PM_NATIVE && pm != PM_SPLIT2 && pm != PM_F64) || (pm != PM_NATIVE && sizeof(T) != 4) ||
      (pm == PM_F64 && !partial64))
    return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 4) {
    if (pm == PM_F64) {
      dim3 grid((unsigned)(((N + 63) / 64) * ((J + 63) / 64)) * n_split, 1, G);
      k_gemm_dw<T, 2, 2, 1, 2, 2, PM_F64><<<grid, 256, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial,
                                                              pdb, n_split, rows_per_split, partial64);
      return hipGetLastError();
    }
    if (pm != PM_NATIVE) {
#define PIGAN_DW_PM(WM_, WN_, NT_, NTH_, BT_)                                                                     \
  do {                                                                                                           \
    dim3 grid((unsigned)(((N + BT_ - 1) / BT_) * ((J + BT_ - 1) / BT_)) * n_split, 1, G);                         \
    k_gemm_dw<T, WM_, WN_, NT_, 2, 4, PM_SPLIT2><<<grid, NTH_, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, \
                                                                       partial, pdb, n_split, rows_per_split,     \
                                                                       partial64);                                \
  } while (0)
      if (N >= 256 && J >= 256) {
        // 256 x 256, 16 waves of 64 x 64 (the fastest measured at 1024 x 1024)
        dim3 grid((unsigned)(((N + 255) / 256) * ((J + 255) / 256)) * n_split, 1, G);
        k_gemm_dw<T, 4, 4, 2, 1, 2, PM_SPLIT2><<<grid, 1024, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J,
                                                                     partial, pdb, n_split, rows_per_split,
                                                                     partial64);
      } else if (N >= 128 && J >= 128) PIGAN_DW_PM(2, 2, 2, 256, 128);
      else if (N >= 64 && J >= 64) PIGAN_DW_PM(2, 2, 1, 256, 64);
      else PIGAN_DW_PM(1, 1, 1, 64, 32);
#undef PIGAN_DW_PM
      return hipGetLastError();
    }
  }
  if constexpr (sizeof(T) == 2) {
    // operand stages straight into an LDS ring; 64 x 64 columns per wave.
    // Block shapes per width are the fastest measured.
    if (N >= 512 && J >= 512) {
      // 256 x 256, 16 waves, 2-stage ring
      dim3 grid((unsigned)(((N + 255) / 256) * ((J + 255) / 256)) * n_split, 1, G);
      k_gemm_dw_tr<T, 4, 4, 2, 4, 2, 1><<<grid, 1024, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial,
                                                              pdb, n_split, rows_per_split);
    } else if (N >= 128 && J >= 256) {
      // 128 x 256, 8 waves, 3-stage ring
      dim3 grid((unsigned)(((N + 127) / 128) * ((J + 255) / 256)) * n_split, 1, G);
      k_gemm_dw_tr<T, 2, 4, 2, 4, 3, 1><<<grid, 512, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial,
                                                             pdb, n_split, rows_per_split);
    } else if (N >= 128 && J >= 128) {
      // 128 x 128, 4 waves, 3-stage ring
      dim3 grid((unsigned)(((N + 127) / 128) * ((J + 127) / 128)) * n_split, 1, G);
      k_gemm_dw_tr<T, 2, 2, 2, 4, 3><<<grid, 256, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial, pdb,
                                                          n_split, rows_per_split);
    } else if (N >= 64 && J >= 64) {
      dim3 grid((unsigned)(((N + 63) / 64) * ((J + 63) / 64)) * n_split, 1, G);
      k_gemm_dw_tr<T, 2, 2, 1, 4><<<grid, 256, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial, pdb,
                                                       n_split, rows_per_split);
    } else {
      dim3 grid((unsigned)(((N + 31) / 32) * ((J + 31) / 32)) * n_split, 1, G);
      k_gemm_dw_tr<T, 1, 1, 1, 4><<<grid, 64, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial, pdb,
                                                      n_split, rows_per_split);
    }
    return hipGetLastError();
  }
  if (N >= 128 && J >= 128) {
    dim3 grid((unsigned)(((N + 127) / 128) * ((J + 127) / 128)) * n_split, 1, G);
    k_gemm_dw<T, 2, 2, 2, 2, 4><<<grid, 256, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial, pdb,
                                                    n_split, rows_per_split, nullptr);
  } else if (N >= 64 && J >= 64) {
    dim3 grid((unsigned)(((N + 63) / 64) * ((J + 63) / 64)) * n_split, 1, G);
    k_gemm_dw<T, 2, 2, 1, 2, 4><<<grid, 256, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial, pdb,
                                                 n_split, rows_per_split, nullptr);
  } else {
    dim3 grid((unsigned)(((N + 31) / 32) * ((J + 31) / 32)) * n_split, 1, G);
    k_gemm_dw<T, 1, 1, 1, 2, 4><<<grid, 64, 0, st>>>(dA, a_g, lda, H, h_g, ldh, R, n_value, N, J, partial, pdb,
                                                n_split, rows_per_split, nullptr);
  }
  return hipGetLastError();
}

#define PIGAN_INST(T)                                                                                    \
  template hipError_t launch_gemm_nt<T>(int, int, int, const NtArgs<T>&, int, hipStream_t);              \
  template hipError_t launch_gemm_dw<T>(const T*, int64_t, int64_t, const T*, int64_t, int64_t, int64_t, \
                                        int64_t, int, int, float*, double*, int, int64_t, int, hipStream_t, int, \
                                        double*);
PIGAN_INST(float)
PIGAN_INST(bf16)
PIGAN_INST(f16)
#undef PIGAN_INST

}  // namespace pigan
