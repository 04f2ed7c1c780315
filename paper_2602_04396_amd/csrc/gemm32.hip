// Grouped GEMM for the subspace refresh: range-finder products (any shape and alignment), Gram matrices,
// blocked Cholesky panels, the inverse of the factor and its application, and the moment rotation.
// One launch runs a list of independent problems (one per weight matrix); a tile table maps each
// workgroup to (problem, tile, K slice).  Operands are addressed by element strides, so any transpose
// and the bf16 gradient type are handled by the loader; accumulation is fp32.  Arithmetic: operands are read in vectors of four
// elements, aligned or not (GemmMode), split into bf16 terms (three per fp32 operand: as exact as fp32) and multiplied on
// v_mfma_f32_32x32x16_bf16; operands too short for a vector, and unaligned ones of the initial projection and of steps with fp32
// gradients, whose bits stay, run on the fp32 matrix cores
// (v_mfma_f32_32x32x2_f32).  k_gemm_planes is the kernel for products of a tall fp32 matrix with a block that many row tiles
// share: the same arithmetic with the block split once (k_pack_planes).
#include "common.h"

namespace lordo {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TK = 32;

#define GAS __attribute__((address_space(1)))

__device__ __forceinline__ const char* resolve(const DevCtx& d, const OpRef& r, int mat) {
  if (r.ext >= 0) return reinterpret_cast<const char*>(ext_ptr(d, r.ext, mat)) + r.off;
  return d.arena + r.off;
}

// One operand of a workgroup tile: X(i, k), i < LIM (the M or N side), k < kend, at base + i*s_i + k*s_k.
// The tile is TMN x TK; a thread fetches NV vectors of four elements along the unit-stride direction
// (scalar accesses where there are fewer than four) and later writes them to LDS as
// S[k][i], the order the matrix-core operands are read in.
template <int TMN, int NV>
struct Operand {
  const char* base;
  int64_t s_i, s_k;
  int is_bf16, lim, kend, i0;
  bool kfast, vec_ok, four_ok;      // four_ok: unit stride over four elements at least, so that a vector can be read at any alignment

  __device__ __forceinline__ void setup(const char* b, int64_t si, int64_t sk, int bf, int lim_, int kend_, int i0_, int kbeg) {
    base = b; s_i = si; s_k = sk; is_bf16 = bf; lim = lim_; kend = kend_; i0 = i0_;
    kfast = sk == 1 && si != 1;
    const int64_t s_fast = kfast ? sk : si, s_slow = kfast ? si : sk;
    const int n_fast = kfast ? kend_ : lim_;
    const uintptr_t align = is_bf16 ? 7 : 15;
    // whole vectors only: every vector then lies entirely inside or entirely outside the operand
    vec_ok = s_fast == 1 && (s_slow & 3) == 0 && (n_fast & 3) == 0 && (reinterpret_cast<uintptr_t>(b) & align) == 0 && (kbeg & 3) == 0;
    four_ok = s_fast == 1 && n_fast >= 4;
  }
  __device__ __forceinline__ void coords(int v, int& ii, int& kk) const {
    if (kfast) { kk = (v % (TK / 4)) * 4; ii = v / (TK / 4); }
    else { ii = (v % (TMN / 4)) * 4; kk = v / (TMN / 4); }
  }
  // Branch-free: an element outside the operand is read from element 0 (always valid) and replaced
  // by zero when the tile is written to LDS.  fetch_raw only issues the loads and leaves the loaded
  // bits untouched, so nothing waits for them until stash() runs one K step later.
  // V4: in vectors at the alignment of an element, those that would run over the end read further back (as OperandBF does)
  template <bool BF16, bool V4>
  __device__ __forceinline__ void fetch_raw(u32x4 (&raw)[NV], int k0, int tid) const {
    const int64_t e_step = kfast ? s_k : s_i;                        // from one element of a vector to the next
    const int d_i = kfast ? 0 : 1, d_k = kfast ? 1 : 0;
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      int ii, kk;
      coords(tid + n * 256, ii, kk);
      const int gi = i0 + ii, gk = k0 + kk;
      if constexpr (V4) {
        const int li = kfast ? lim - 1 : lim - 4, lk = kfast ? kend - 4 : kend - 1;
        const int64_t at = (int64_t)(gi < li ? gi : li) * s_i + (int64_t)(gk < lk ? gk : lk) * s_k;
        typedef u32x2 half_t __attribute__((aligned(2)));
        typedef u32x4 full_t __attribute__((aligned(4)));
        if constexpr (BF16) {
          const u32x2 w = *(const GAS half_t*)((const GAS char*)base + at * 2);
          raw[n].x = w.x; raw[n].y = w.y;
        } else {
          raw[n] = *(const GAS full_t*)((const GAS char*)base + at * 4);
        }
        continue;
      }
      const int64_t idx = (int64_t)gi * s_i + (int64_t)gk * s_k;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = gi + e * d_i < lim && gk + e * d_k < kend;
        const int64_t at = ok ? idx + e * e_step : 0;
        if constexpr (BF16) raw[n][e] = *reinterpret_cast<const GAS uint16_t*>((const GAS char*)base + at * 2);
        else raw[n][e] = *reinterpret_cast<const GAS uint32_t*>((const GAS char*)base + at * 4);
      }
    }
  }
  // Writes the tile starting at k0 to S[k][i], zeros past the end of k.  Rows past the last one stay what was read in their place: they
  // end in elements of C that are not stored.
  template <bool BF16, bool V4>
  __device__ __forceinline__ void stash(const u32x4 (&raw)[NV], float (*S)[TMN + 4], int k0, int tid) const {
    if (k0 + TK > kend || (V4 && !kfast && i0 + TMN > lim)) put<BF16, V4, true>(raw, S, k0, tid);      // (uniform)
    else put<BF16, V4, false>(raw, S, k0, tid);
  }
  template <bool BF16, bool V4, bool EDGE>
  __device__ __forceinline__ void put(const u32x4 (&raw)[NV], float (*S)[TMN + 4], int k0, int tid) const {
    const int d_k = kfast ? 1 : 0;
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      int ii, kk;
      coords(tid + n * 256, ii, kk);
      const int gi = i0 + ii, gk = k0 + kk;
      u32x4 x = raw[n];
      if constexpr (V4) {
        if constexpr (BF16) x = u32x4{x.x << 16, x.x & 0xffff0000u, x.y << 16, x.y & 0xffff0000u};
        if constexpr (EDGE) {              // a vector that would run over the end was read further back
          const int past = kfast ? gk + 4 - kend : gi + 4 - lim, over = past > 0 && past < 4 ? past : 0;
          x = (over & 1) ? u32x4{x.y, x.z, x.w, 0u} : x;
          x = (over & 2) ? u32x4{x.z, x.w, 0u, 0u} : x;
        }
      } else if constexpr (BF16) {
        x = u32x4{x.x << 16, x.y << 16, x.z << 16, x.w << 16};
      }
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = __uint_as_float(EDGE && gk + e * d_k >= kend ? 0u : x[e]);
      if (kfast) {
#pragma unroll
        for (int e = 0; e < 4; ++e) S[kk + e][ii] = r[e];
      } else {
        *reinterpret_cast<f32x4*>(&S[kk][ii]) = r;
      }
    }
  }
};

// K loop of one workgroup tile on the fp32 matrix cores, specialised on the element type of A.
template <int WB, bool A_BF16, bool V4, int TM, int NV>
__device__ __forceinline__ void gemm_loop(f32x16 (&acc)[WB][WB], const Operand<TM, NV>& opA, const Operand<TM, NV>& opB,
                                          float (*As)[TM + 4], float (*Bs)[TM + 4], int kbeg, int K, int tid, int lane, int wm, int wn) {
  u32x4 ra[NV], rb[NV];
  opA.template fetch_raw<A_BF16, V4>(ra, kbeg, tid);
  opB.template fetch_raw<false, V4>(rb, kbeg, tid);
  for (int k0 = kbeg; k0 < K; k0 += TK) {
    __syncthreads();                           // previous tile fully consumed
    opA.template stash<A_BF16, V4>(ra, As, k0, tid);
    opB.template stash<false, V4>(rb, Bs, k0, tid);
    __syncthreads();
    if (k0 + TK < K) {
      opA.template fetch_raw<A_BF16, V4>(ra, k0 + TK, tid);
      opB.template fetch_raw<false, V4>(rb, k0 + TK, tid);
    }
    asm volatile("" ::: "memory");             // keep the loads above the arithmetic: they must be in flight during it
#pragma unroll
    for (int kk = 0; kk < TK; kk += 2) {
      float av[WB], bv[WB];
#pragma unroll
      for (int a = 0; a < WB; ++a) av[a] = As[kk + (lane >> 5)][wm + 32 * a + (lane & 31)];
#pragma unroll
      for (int b = 0; b < WB; ++b) bv[b] = Bs[kk + (lane >> 5)][wn + 32 * b + (lane & 31)];
#pragma unroll
      for (int a = 0; a < WB; ++a)
#pragma unroll
        for (int b = 0; b < WB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Split-bf16 variant of the K loop for the range-finder products (Alg. 2 sketch and power
// iteration).  Operands go to LDS as bf16 planes in matrix-core fragment order -- a bf16 source is
// exact, an fp32 operand becomes hi + mid + lo, each rounded to nearest (2^-26 relative, as exact as fp32) -- and the
// products run on v_mfma_f32_32x32x16_bf16: three passes for a bf16 source, six for an fp32 one
// (all products of terms down to 2^-24).  Two terms (2^-16) are not enough: the trailing directions
// of the range finder's block sit in the noise of the source, where gaps between singular values are
// of the order of a percent, and a 2^-16 perturbation moved the subspace by up to 9e-4 in Frobenius
// norm of the projector, against 3e-5 for fp32 arithmetic.
// Plane element (i, k) of a TMN x 32 tile: (i/32) * FRAG_BLOCK + (k/8) * 264 + (i%32)*8 + k%8 (eight elements
// of padding per 32 x 8 group and eight more per 32 x 32 block).  The 8-byte writes of a wave then meet at most twice in a bank,
// the least there is: the lanes of a transposed patch lie four rows (64 bytes) apart, eight to a block, so the blocks have to be
// 16 bytes off (they met eight times without), and rows contiguous in k are dealt out four apart (four times).  28 matrices,
// r = 512, 4096 .. 11008 rows: Gram matrices 674 -> 476 us, R = Q_new^T Q 862 -> 611 us; 72 matrices of 768 .. 3072, r = 128: 48 -> 41 us.
// ---------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int FRAG_BLOCK = 4 * 264 + 8;      // elements per 32 x 32 block
__device__ __forceinline__ int frag_index(int i, int k) { return (i >> 5) * FRAG_BLOCK + (k >> 3) * 264 + (i & 31) * 8 + (k & 7); }

// Operand tile of the split-bf16 loop, read in vectors of four elements along the unit-stride direction.  UA = false: every
// vector is aligned and lies entirely inside or outside the operand.  UA = true (rows of an odd number of elements, pointers into
// the middle of a vector, ranks that are no multiple of four): vectors are read at the alignment of an element, and one that would run
// over the end of the operand is read further back, ending with its last element; shift_in() then moves the elements to their
// places and zeros in behind them (a uniform branch: only tiles at the end have such vectors).  On the fp32 matrix cores with
// element accesses, which such operands took before, a refresh of 21 matrices (2047 x 2047 .. 5001, r = 171) took 6.25 ms from bf16 and
// 6.23 ms from fp32, so 3.11 and 3.68 ms.
// A thread owns NV vectors of four elements.  KF (k is the unit-stride direction): they pack directly; else they are a patch of
// four i and NV consecutive k, which the thread transposes in registers.
// Addresses: a uniform base that moves on with k and one 32-bit byte offset per vector, fixed over the loop (every array is below
// 4 GiB); only the last K tile works its offsets out again, so that nothing past the end is read.
template <int TMN, bool UA, bool BF16, bool KF>
struct OperandBF {
  static constexpr int ES = BF16 ? 2 : 4;
  static constexpr int NV = TMN / 32;
  const GAS char* base;
  int64_t k_bytes;                              // from one k to the next
  int lim, kend, i0, kk0;                       // kk0: k of the thread's first vector inside a K tile
  uint32_t off[NV];                             // vector n at K tile 0

  __device__ __forceinline__ void setup(const char* b, int64_t s_i, int64_t s_k, int lim_, int kend_, int i0_, int tid) {
    base = (const GAS char*)b; lim = lim_; kend = kend_; i0 = i0_;
    k_bytes = s_k * ES;
    kk0 = KF ? (tid & 7) * 4 : tid / (TMN / 4) * NV;
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      int gi = i0 + row(n, tid);                // rows past the end are read from the last one, vectors across it further back
      const int last = KF ? lim - 1 : lim - 4;
      gi = gi < last ? gi : last;
      off[n] = (uint32_t)gi * (uint32_t)(s_i * ES) + (uint32_t)(kk0 + (KF ? 0 : n)) * (uint32_t)k_bytes;
    }
  }
  // first i of vector n inside the tile (along i: of the whole patch)
  static __device__ __forceinline__ int row(int n, int tid) {
    return KF ? n * 32 + ((tid >> 1) & 28) + (tid >> 6)                    // the eight rows of a wave lie four apart
              : tid % (TMN / 4) * 4;
  }
  __device__ __forceinline__ void fetch(u32x4 (&raw)[NV], int k0) const {
    const bool whole = k0 + TK <= kend;
    const GAS char* at = whole ? base + (int64_t)k0 * k_bytes : base;
    uint32_t o[NV];
#pragma unroll
    for (int n = 0; n < NV; ++n) o[n] = off[n];
    if (!whole) {
#pragma unroll
      for (int n = 0; n < NV; ++n) {
        const int kk = kk0 + (KF ? 0 : n), last = kend - (KF ? 4 : 1);
        const int k = k0 + kk < last ? k0 + kk : last;
        o[n] += (uint32_t)(k - kk) * (uint32_t)k_bytes;
      }
    }
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      typedef u32x2 half_t __attribute__((aligned(2)));
      typedef u32x4 full_t __attribute__((aligned(4)));
      if constexpr (BF16) {
        u32x2 w;
        if constexpr (UA) w = *(const GAS half_t*)(at + o[n]);
        else w = *(const GAS u32x2*)(at + o[n]);
        raw[n].x = w.x; raw[n].y = w.y;
      } else if constexpr (UA) {
        raw[n] = *(const GAS full_t*)(at + o[n]);
      } else {
        raw[n] = *(const GAS u32x4*)(at + o[n]);
      }
    }
  }
  // Elements past the end of a vector that starts inside (at `at`, of `end`): so many it was read too far back
  static __device__ __forceinline__ int past_end(int at, int end) { return at < end && at + 4 > end ? at + 4 - end : 0; }
  static __device__ __forceinline__ u32x4 shift_in(u32x4 x, int n) {
    if constexpr (BF16) {
      const uint64_t v = (((uint64_t)x.y << 32) | x.x) >> (16 * n);
      x.x = (uint32_t)v; x.y = (uint32_t)(v >> 32);
    } else {
      if (n & 1) x = u32x4{x.y, x.z, x.w, 0u};
      if (n & 2) x = u32x4{x.z, x.w, 0u, 0u};
    }
    return x;
  }
  // Two fp32 values -> three packed bf16 pairs whose sum is the values to 2^-26: hi is the value rounded to nearest,
  // mid the (exactly representable) remainder rounded to nearest, lo the rounded rest; the conversion is the
  // hardware's packed round-to-nearest-even instruction, about five vector operations per element.
  // Rounding to nearest, not truncation: truncated terms all carry the sign of the value, so on the diagonal of a
  // Gram matrix X^T X every cross product hi * lo is positive; those below half an ulp of the running sum are
  // rounded away one k-step after the other, and the diagonal came out too small by up to 2e-5 relative (growing
  // with the length of the contraction), i.e. the columns of the orthonormalised block too long by 1e-5.  With
  // terms of random sign the same loss has zero mean.
  static __device__ __forceinline__ uint32_t pack_rne(float x0, float x1) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {x0, x1};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  }
  static __device__ __forceinline__ void split3(uint32_t x0, uint32_t x1, uint32_t (&t)[3]) {
    const float f0 = __uint_as_float(x0), f1 = __uint_as_float(x1);
    t[0] = pack_rne(f0, f1);
    const float r0 = f0 - __uint_as_float(t[0] << 16);
    const float r1 = f1 - __uint_as_float(t[0] & 0xffff0000u);
    t[1] = pack_rne(r0, r1);
    const float s0 = r0 - __uint_as_float(t[1] << 16);
    const float s1 = r1 - __uint_as_float(t[1] & 0xffff0000u);
    t[2] = pack_rne(s0, s1);
  }
  // P: the operand's planes (one for an exact bf16 operand, three for an fp32 one), `plane` elements apart
  __device__ __forceinline__ void stash(u32x4 (&raw)[NV], uint16_t* P, int plane, int k0, int tid) const {
    // Rows past the last one stay what was read in their place: they end in elements of C that are not stored.  What lies past the end of
    // k becomes zero.  (Uniform branches, selects inside them.  Zeros for the rows too, by lane branches in every K step of an edge tile:
    // 48 x (5824 x 320 and 160 x 928), r = 136, fp32 gradients 850 us a step, 716 so.)
    if constexpr (UA && !KF) {
      if (i0 + TMN > lim) {
#pragma unroll
        for (int n = 0; n < NV; ++n) raw[n] = shift_in(raw[n], past_end(i0 + row(n, tid), lim));
      }
    }
    if (k0 + TK > kend) {
#pragma unroll
      for (int n = 0; n < NV; ++n) {
        const int k = k0 + kk0 + (KF ? 0 : n);
        if constexpr (UA && KF) raw[n] = shift_in(raw[n], past_end(k, kend));
        const uint32_t keep = k < kend ? 0xffffffffu : 0u;
#pragma unroll
        for (int e = 0; e < (BF16 ? 2 : 4); ++e) raw[n][e] &= keep;
      }
    }
    if constexpr (KF) {
#pragma unroll
      for (int n = 0; n < NV; ++n) {
        const int at = frag_index(row(n, tid), kk0);          // four consecutive k: 8 contiguous bytes
        if constexpr (BF16) {
          *reinterpret_cast<u32x2*>(P + at) = u32x2{raw[n].x, raw[n].y};
        } else {
          uint32_t ta[3], tb[3];
          split3(raw[n].x, raw[n].y, ta);
          split3(raw[n].z, raw[n].w, tb);
#pragma unroll
          for (int c = 0; c < 3; ++c) *reinterpret_cast<u32x2*>(P + c * plane + at) = u32x2{ta[c], tb[c]};
        }
      }
    } else {
      // vector n holds i = ii .. ii+3 at k = kk0 + n; row ii + e of the plane gets k = kk0 .. kk0 + NV - 1
      const int ii = row(0, tid);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int at = frag_index(ii + e, kk0);
        uint32_t t[NV / 2][3];
#pragma unroll
        for (int h = 0; h < NV / 2; ++h) {
          if constexpr (BF16) {                               // element e of vector n: half (e & 1) of word e / 2
            t[h][0] = __builtin_amdgcn_perm(raw[2 * h + 1][e >> 1], raw[2 * h][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
          } else {
            split3(raw[2 * h][e], raw[2 * h + 1][e], t[h]);
          }
        }
#pragma unroll
        for (int c = 0; c < (BF16 ? 1 : 3); ++c) {
          if constexpr (NV == 4) *reinterpret_cast<u32x2*>(P + c * plane + at) = u32x2{t[0][c], t[1][c]};
          else *reinterpret_cast<uint32_t*>(P + c * plane + at) = t[0][c];
        }
      }
    }
  }
};

// same_ab (uniform): the tile of B is the tile of A (a diagonal tile of a Gram matrix X^T X): it is fetched and
// split once and the B fragments are read from the planes of A.
// DIAG: such a tile also sums the squares of its columns in double, from the values as they pass through its registers, and leaves them
// at g.diag (or, not split, as the diagonal of C).  The products of the two middle terms are dropped from the six: squares on the
// diagonal, always positive and about 2^-18 of the entry; in a long contraction they fall below half an ulp of the running sum and
// are rounded away step after step.  The diagonal came out 2e-6 to 3e-6 too small at p >= 4096 and the columns of the orthonormalised
// block that much too long: 7e-5 in || Q^T Q - I ||_F at r = 512.  The diagonal carries the column norms, so it alone is summed exactly.
// (As passes of their own, over X and over partial sums, with a launch for the diagonal shift, 24 us behind every Gram matrix of the
// 125M set: its refresh 1897 -> 1796 us; four blocks of 7B 17.99 -> 17.39 ms, two blocks of 125M
// 641 -> 615 us.)
template <int WB, bool UA, bool A_BF16, bool A_KF, bool B_KF, bool DIAG = false>
__device__ __forceinline__ void gemm_loop_bf(f32x16 (&acc)[WB][WB], const GemmDesc& g, const char* baseA, const char* baseB,
                                             uint16_t* lds, int m0, int n0, int kbeg, int K, int tid, int lane, int wm, int wn, bool same_ab,
                                             char* arena, int slice) {
  constexpr int TM = 64 * WB;
  typedef OperandBF<TM, UA, A_BF16, A_KF> OpA;
  typedef OperandBF<TM, UA, false, B_KF> OpB;
  OpA opA;
  OpB opB;
  opA.setup(baseA, g.sAm, g.sAk, g.M, K, m0, tid);
  opB.setup(baseB, g.sBn, g.sBk, g.N, K, n0, tid);
  constexpr int PLANE = (TM / 32) * FRAG_BLOCK;                   // elements
  constexpr int NA = A_BF16 ? 1 : 3;                           // planes of A; B always has three
  uint16_t* PA = lds;
  uint16_t* PB = (!A_BF16 && same_ab) ? lds : lds + NA * PLANE;
  const bool own_b = !DIAG && (A_BF16 || !same_ab);
  double dsum[4] = {0.0, 0.0, 0.0, 0.0};                       // DIAG: of the thread's four columns over its rows
  auto step = [&](u32x4 (&ra)[OpA::NV], u32x4 (&rb)[OpB::NV], int k0) {
    __syncthreads();                           // previous tile fully consumed
    opA.stash(ra, PA, PLANE, k0, tid);
    if (own_b) opB.stash(rb, PB, PLANE, k0, tid);
    if constexpr (DIAG) {
#pragma unroll
      for (int n = 0; n < OpA::NV; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double x = (double)__uint_as_float(ra[n][e]);
          dsum[e] = fma(x, x, dsum[e]);
        }
    }
    __syncthreads();
    opA.fetch(ra, k0 + 2 * TK);                // (past the end: the last vectors once more, so that every step has the same loads in flight)
    if (own_b) opB.fetch(rb, k0 + 2 * TK);
    asm volatile("" ::: "memory");             // keep the loads above the arithmetic: they must be in flight during it
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 fa[NA][WB], fb[3][WB];
      const int kg = 16 * ks + 8 * (lane >> 5);
#pragma unroll
      for (int a = 0; a < WB; ++a) {
        const int at = frag_index(wm + 32 * a + (lane & 31), kg);
#pragma unroll
        for (int c = 0; c < NA; ++c) fa[c][a] = *reinterpret_cast<const bf16x8*>(PA + c * PLANE + at);
      }
#pragma unroll
      for (int b = 0; b < WB; ++b) {
        const int at = frag_index(wn + 32 * b + (lane & 31), kg);
#pragma unroll
        for (int c = 0; c < 3; ++c) fb[c][b] = *reinterpret_cast<const bf16x8*>(PB + c * PLANE + at);
      }
      // every product of terms down to 2^-24: (a0, b0..b2) for an exact A; plus (a1, b0), (a1, b1), (a2, b0)
#pragma unroll
      for (int ca = 0; ca < NA; ++ca)
#pragma unroll
        for (int cb = 0; cb + ca < 3; ++cb)
#pragma unroll
          for (int a = 0; a < WB; ++a)
#pragma unroll
            for (int b = 0; b < WB; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ca][a], fb[cb][b], acc[a][b], 0, 0, 0);
    }
  };
  // Two K tiles in flight, in register sets that alternate statically: the load of a K tile has a whole step more to arrive.  With one in
  // flight and 64-bit addresses of every vector in every step a tile's K step was a memory latency: one 256 x 256 matrix with fp32
  // gradients (4 tiles, 8 steps) 16.1 -> 11.7 us, 18 matrices 957 x 957 .. 2201, r = 39, Y = Src B 126 -> 62 us, 6 of 2304 x 2304 .. 6400,
  // r = 384, fp32 gradients 606 -> 466 us; full launches of 128-wide tiles are as fast as before.
  u32x4 ra0[OpA::NV], rb0[OpB::NV], ra1[OpA::NV], rb1[OpB::NV];
  opA.fetch(ra0, kbeg);
  if (own_b) opB.fetch(rb0, kbeg);
  opA.fetch(ra1, kbeg + TK);
  if (own_b) opB.fetch(rb1, kbeg + TK);
  int k0 = kbeg;
  for (; k0 + TK < K; k0 += 2 * TK) {
    step(ra0, rb0, k0);
    step(ra1, rb1, k0 + TK);
  }
  if (k0 < K) step(ra0, rb0, k0);
  if constexpr (DIAG) {
    static_assert(!A_BF16 && !A_KF, "patches of four columns");
    constexpr int GROUPS = 1024 / TM;                          // threads that share four columns, added in their order
    double (*red)[TM] = reinterpret_cast<double (*)[TM]>(lds);
    static_assert(sizeof(double) * GROUPS * TM <= sizeof(uint16_t) * 3 * PLANE, "partial sums must fit");
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) red[tid / (TM / 4)][opA.row(0, tid) + e] = dsum[e];
    __syncthreads();
    const int col = m0 + tid;
    if (tid < TM && col < g.M) {
      double sum = 0.0;
#pragma unroll
      for (int i = 0; i < GROUPS; ++i) sum += red[i][tid];
      if (g.ksplit > 1) *((GAS double*)(arena + g.diag) + (int64_t)slice * g.M + col) = sum;
      else *((GAS float*)(arena + g.C.off) + (int64_t)col * g.ldc + col) = (float)sum;
    }
  }
}

// The loop for the unit-stride directions of a problem's operands (uniform).  A bf16 A is a source or a gradient, whose B (start block, Y, Z, Q)
// is never contiguous in k.  WITH_DIAG: problems may carry g.diag.
template <int WB, bool UA, bool A_BF16, bool WITH_DIAG>
__device__ __forceinline__ void gemm_loops_bf(f32x16 (&acc)[WB][WB], const GemmDesc& g, const char* baseA, const char* baseB, uint16_t* lds,
                                              int m0, int n0, int kbeg, int K, int tid, int lane, int wm, int wn, bool same_ab,
                                             char* arena, int slice) {
  const bool akf = g.sAk == 1 && g.sAm != 1, bkf = g.sBk == 1 && g.sBn != 1;
  if constexpr (!A_BF16 && WITH_DIAG) {
    if (same_ab && g.diag >= 0 && !akf && !bkf) {
      gemm_loop_bf<WB, UA, false, false, false, true>(acc, g, baseA, baseB, lds, m0, n0, kbeg, K, tid, lane, wm, wn, true, arena, slice);
      return;
    }
  }
  if constexpr (!A_BF16) {
    if (bkf) {
      if (akf) gemm_loop_bf<WB, UA, A_BF16, true, true>(acc, g, baseA, baseB, lds, m0, n0, kbeg, K, tid, lane, wm, wn, same_ab, arena, slice);
      else gemm_loop_bf<WB, UA, A_BF16, false, true>(acc, g, baseA, baseB, lds, m0, n0, kbeg, K, tid, lane, wm, wn, same_ab, arena, slice);
      return;
    }
  }
  if (akf) gemm_loop_bf<WB, UA, A_BF16, true, false>(acc, g, baseA, baseB, lds, m0, n0, kbeg, K, tid, lane, wm, wn, same_ab, arena, slice);
  else gemm_loop_bf<WB, UA, A_BF16, false, false>(acc, g, baseA, baseB, lds, m0, n0, kbeg, K, tid, lane, wm, wn, same_ab, arena, slice);
}

// 256 threads = 4 waves in a 2 x 2 grid; each wave WB x WB accumulator blocks of 32 x 32, so the
// workgroup tile is 64*WB square (64 for small problems, 128 for large launches).  The next K tile
// is fetched into registers while the matrix cores work on the one in LDS.
// MODE (GemmMode; known on the host for a whole launch): how the operands of all its problems can be read.  One kernel that chose per tile
// held six loops in the registers of the largest.  A_BF16 matters in the first two modes, src_is_bf16 in the third.
template <int WB, int MODE, bool A_BF16>
__global__ __launch_bounds__(256, MODE == GEMM_RAGGED ? 2 : MODE == GEMM_ANY && WB == 1 ? 4 : 1) void k_gemm32(DevCtx d, const GemmDesc* __restrict__ descs,
                                                const GemmTile* __restrict__ tiles, int src_is_bf16, float alpha_mul, int sub_m, int sub_n) {
  constexpr int TM = 64 * WB, TN = 64 * WB;
  constexpr int PITCH = TM + 4;
  constexpr int NV = TM * TK / 4 / 256;
  const GemmTile t = tiles[blockIdx.x];
  const GemmDesc g = descs[t.desc];
  if (mat_skipped(d, g.mat)) return;
  const int M = g.M, N = g.N;
  const int kbeg = g.ksplit > 1 ? t.ks * g.klen : 0;
  int K = g.ksplit > 1 ? (kbeg + g.klen < g.K ? kbeg + g.klen : g.K) : g.K;           // end of this slice
  // a table entry covers sub_m x sub_n tiles of this kernel (1 x 1 but where the table was made for k_gemm_planes)
  const int m0 = (t.tm * sub_m + (int)blockIdx.y) * TM, n0 = (t.tn * sub_n + (int)blockIdx.z) * TN;
  if (sub_m + sub_n > 2 && (m0 >= M || n0 >= N)) return;
  if (g.tri && n0 + TN < K) K = n0 + TN;            // B is zero below this tile's last column
  float* C = reinterpret_cast<float*>(const_cast<char*>(resolve(d, g.C, g.mat)));
  float* C2 = g.C2.off >= 0 ? reinterpret_cast<float*>(const_cast<char*>(resolve(d, g.C2, g.mat))) : nullptr;

  // As | Bs of the fp32 loop, or up to six bf16 planes of the split loop
  constexpr int PLANE_FLOATS = (MODE != GEMM_ANY && A_BF16 ? 4 : 6) * (TM / 32) * FRAG_BLOCK / 2;
  constexpr int LDS_FLOATS = MODE == GEMM_ANY && 2 * TK * PITCH > PLANE_FLOATS ? 2 * TK * PITCH : PLANE_FLOATS;
  __shared__ __attribute__((aligned(16))) float lds_raw[LDS_FLOATS];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave & 1) * 32 * WB, wn = (wave >> 1) * 32 * WB;

  f32x16 acc[WB][WB];
#pragma unroll
  for (int a = 0; a < WB; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  const char* baseA = resolve(d, g.A, g.mat);
  const char* baseB = resolve(d, g.B, g.mat);
  // same matrix, same strides with the roles of the two indices swapped, same tile: A(m, k) = B(k, n = m)
  const bool same_ab = g.A.off == g.B.off && g.A.ext == g.B.ext && g.sAm == g.sBn && g.sAk == g.sBk && m0 == n0 && M == N;
  uint16_t* planes = reinterpret_cast<uint16_t*>(lds_raw);
  if constexpr (MODE != GEMM_ANY) {
    if (kbeg < K) gemm_loops_bf<WB, MODE == GEMM_RAGGED, A_BF16, true>(acc, g, baseA, baseB, planes, m0, n0, kbeg, K, tid, lane, wm, wn, !A_BF16 && same_ab, d.arena, t.ks);
  } else {
    const int a_bf16 = g.a_bf16 == 2 ? src_is_bf16 : g.a_bf16;
    float (*As)[PITCH] = reinterpret_cast<float (*)[PITCH]>(lds_raw);
    float (*Bs)[PITCH] = reinterpret_cast<float (*)[PITCH]>(lds_raw + TK * PITCH);
    Operand<TM, NV> opA, opB;
    opA.setup(baseA, g.sAm, g.sAk, a_bf16, M, K, m0, kbeg);
    opB.setup(baseB, g.sBn, g.sBk, 0, N, K, n0, kbeg);
    const bool vec = opA.vec_ok && opB.vec_ok;
    if (kbeg >= K) {
    } else if (vec) {
      if (a_bf16) gemm_loops_bf<WB, false, true, false>(acc, g, baseA, baseB, planes, m0, n0, kbeg, K, tid, lane, wm, wn, false, d.arena, t.ks);
      else gemm_loops_bf<WB, false, false, false>(acc, g, baseA, baseB, planes, m0, n0, kbeg, K, tid, lane, wm, wn, same_ab, d.arena, t.ks);
    } else if (opA.four_ok && opB.four_ok) {
      if (a_bf16) gemm_loop<WB, true, true>(acc, opA, opB, As, Bs, kbeg, K, tid, lane, wm, wn);
      else gemm_loop<WB, false, true>(acc, opA, opB, As, Bs, kbeg, K, tid, lane, wm, wn);
    } else {
      if (a_bf16) gemm_loop<WB, true, false>(acc, opA, opB, As, Bs, kbeg, K, tid, lane, wm, wn);
      else gemm_loop<WB, false, false>(acc, opA, opB, As, Bs, kbeg, K, tid, lane, wm, wn);
    }
  }

  float* Pp = g.ksplit > 1 ? reinterpret_cast<float*>(const_cast<char*>(resolve(d, g.P, g.mat))) + (int64_t)t.ks * M * N : nullptr;
  // accumulator register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32 of the block
#pragma unroll
  for (int a = 0; a < WB; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b) {
      const int col = n0 + wn + 32 * b + (lane & 31);
      if (col >= N) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        int row = m0 + wm + 32 * a + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (row < M && Pp) {
          Pp[(int64_t)row * N + col] = acc[a][b][v];
        } else if (row < M && !(row == col && MODE != GEMM_ANY && g.diag >= 0)) {
          int64_t o = (int64_t)row * g.ldc + col;
          float val = g.alpha * alpha_mul * acc[a][b][v];
          if (g.beta != 0.f) val = fmaf(g.beta, C[o], val);
          C[o] = val;
          if (C2) C2[o] = val * val;
        }
      }
    }
}

// Sum of the split-K slices in slice order (deterministic), then alpha, beta and the optional square.  Of a Gram matrix the lower
// triangle, which is all that is read, with the diagonal from its own sums.
__global__ __launch_bounds__(256) void k_gemm_reduce(DevCtx d, const GemmDesc* __restrict__ descs) {
  const GemmDesc g = descs[blockIdx.y];
  if (g.ksplit <= 1 || mat_skipped(d, g.mat)) return;
  const float* Pp = reinterpret_cast<const float*>(resolve(d, g.P, g.mat));
  float* C = reinterpret_cast<float*>(const_cast<char*>(resolve(d, g.C, g.mat)));
  float* C2 = g.C2.off >= 0 ? reinterpret_cast<float*>(const_cast<char*>(resolve(d, g.C2, g.mat))) : nullptr;
  const int64_t total = (int64_t)g.M * g.N;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const uint32_t row = (uint32_t)e / (uint32_t)g.N, col = (uint32_t)e - row * (uint32_t)g.N;      // (M N < 2^32: r x r products)
    if (g.diag >= 0 && col >= row) {
      if (col > row) continue;
      const double* part = reinterpret_cast<const double*>(d.arena + g.diag);
      double sum = 0.0;
      for (int sl = 0; sl < g.ksplit; ++sl) sum += part[(int64_t)sl * g.M + row];
      C[(int64_t)row * g.ldc + row] = (float)sum;
      continue;
    }
    float acc = 0.f;
    // eight loads in flight, added in slice order (one at a time, each waited for: 18 us at r = 128, 72 matrices, 15 slices)
    int sl = 0;
    for (; sl + 8 <= g.ksplit; sl += 8) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = Pp[(int64_t)(sl + i) * total + e];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc += x[i];
    }
    for (; sl < g.ksplit; ++sl) acc += Pp[(int64_t)sl * total + e];
    int64_t o = (int64_t)row * g.ldc + col;
    float val = g.alpha * acc;
    if (g.beta != 0.f) val = fmaf(g.beta, C[o], val);
    C[o] = val;
    if (C2) C2[o] = val * val;
  }
}
hipError_t launch_gemm_reduce(const DevCtx& d, const GemmDesc* descs, int ndescs, hipStream_t s) {
  if (ndescs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gemm_reduce, dim3(64, ndescs), dim3(256), 0, s, d, descs);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// C = A B with a tall fp32 A (rows contiguous in k) and a narrow B that many row tiles share: the products of an fp32
// refresh source with a block (Sec. 2 range finder), the application of the factor's inverse, X M^T, and the moment
// rotation.  Same arithmetic, in the same order, as the split loop above (three bf16 terms per operand, six products),
// so the results are the same bits; what differs is who does the splitting.  There, every 128 x 128 tile splits its
// share of B again and stages one K step at a time between two barriers; here B is split once (k_pack_planes) into
// operand fragments that travel from global memory to LDS without passing through registers, and A is split once per
// 128 rows x up to 256 columns.  Four waves in a 2 x 2 grid, wave tile 64 rows x 32 NBW columns; two LDS buffers of
// one k-step of 16 each (72 KiB at NBW = 4: two workgroups per compute unit, one splits while the other multiplies);
// the rows of A are requested two to three k-steps ahead of their use.  The loads into LDS are issued from inline
// assembly with explicit waits: in an even step they precede the loads of A, so "at most the four loads of A
// outstanding" implies that they have landed.
// Measured (24 x 7 matrices, 2048 x 2048 .. 5632, r = 256, fp32 source): Y = Src B 4.6 -> 3.54 ms at edge 128, 3.65 at 256 (3.8 TFLOP of
// bf16 products, 1.07 PFLOP/s; the matrix cores are busy 64 % of the cycles at a clock that this load holds at 1.59 GHz: power is the
// bound, and skipping the zero half of M^T gains nothing), X M^T 0.51 -> 0.33 ms, rotation product 0.51 -> 0.40 ms (both on edge 128;
// profiles/1b_synchronisation_*.txt); 28 matrices of 4096 .. 11008 at r = 512: X M^T 0.48 -> 0.35 and 0.58 -> 0.43 ms; 72 matrices
// of 768 .. 3072 at r = 128, fp32 source: three products 0.29 -> 0.25 ms each.
// ---------------------------------------------------------------------------------------
#define LDS_AS __attribute__((address_space(3)))
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// lane i's 16 bytes land at lds_dst_wave_base + 16 i; M0 carries the LDS address, one wait state before its use
__device__ __forceinline__ void plane_to_lds(const GAS u32x4* src, u32x4* lds_dst_wave_base) {
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(LDS_AS void*)lds_dst_wave_base;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}
#pragma clang diagnostic pop
#define WAIT_VM_BARRIER(N) asm volatile("s_waitcnt vmcnt(" #N ") lgkmcnt(0)\n\ts_barrier" ::: "memory")

template <int NBW, bool ONCE>      // ONCE: A is read by one column tile only (streaming loads)
__global__ __launch_bounds__(256, 2) void k_gemm_planes(DevCtx d, const GemmDesc* __restrict__ descs, const GemmTile* __restrict__ tiles,
                                                        int ntiles, const uint16_t* __restrict__ p0, const uint16_t* __restrict__ p1,
                                                        const uint16_t* __restrict__ p2) {
  constexpr int TN = 64 * NBW;
  constexpr int ASLOTS = 12, BSLOTS = 6 * NBW, SLOTS = ASLOTS + BSLOTS;     // 1 KiB fragments of a k-step: three planes each
  constexpr int BLOADS = (BSLOTS + 3) / 4;                                  // fragments of B a wave brings in per k-step
  // Runs of sixteen consecutive tiles share an XCD and so its L2: sixteen row tiles read the same planes of B
  // (workgroups go to the eight XCDs round-robin by index; whole runs keep uneven matrices spread over all of them).
  const int b = (int)blockIdx.x;
  const int tile = ((b >> 7) * 8 + (b & 7)) * 16 + ((b >> 3) & 15);
  if (tile >= ntiles) return;
  const GemmTile t = tiles[tile];
  const GemmDesc g = descs[t.desc];
  if (mat_skipped(d, g.mat)) return;
  const int M = g.M, N = g.N, m0 = t.tm * 128, n0 = t.tn * TN;
  const int kend = g.tri && n0 + TN < g.K ? n0 + TN : g.K;                   // (tri: B is zero below this tile's last column)
  const int nsteps = (kend + 31) / 32 * 2;
  const int64_t kgroups = pad32(g.K) / 8;
  const int nblocks = (int)pad32(N) / 32;

  extern __shared__ u32x4 lds_planes[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;

  // B fragments: slot (plane, block of 32 columns); a block past the last repeats the last (its columns are not stored)
  const int64_t lr_off = d.mats[g.mat].lr_off;
  const GAS u32x4* bsrc[BLOADS];
  int bslot[BLOADS];
#pragma unroll
  for (int j = 0; j < BLOADS; ++j) {
    const int i = wave + 4 * j < BSLOTS ? wave + 4 * j : BSLOTS - 1;
    const int c = i / (2 * NBW), nb = n0 / 32 + i % (2 * NBW);
    const uint16_t* pl = c == 0 ? p0 : c == 1 ? p1 : p2;
    bsrc[j] = (const GAS u32x4*)(pl + lr_off) + (int64_t)(nb < nblocks ? nb : nblocks - 1) * kgroups * 32 + lane;
    bslot[j] = ASLOTS + i;
  }
  auto issue_b = [&](int s, int buf) {
    s = s < nsteps ? s : nsteps - 1;               // past the end the last step again: the same number of loads in every step
#pragma unroll
    for (int j = 0; j < BLOADS; ++j) plane_to_lds(bsrc[j] + (int64_t)s * 64, lds_planes + (buf * SLOTS + bslot[j]) * 64);
  };
  // A: thread = (row, k octet of a step); a chunk is two steps.  Rows past M repeat row M - 1 and are not stored.
  const int arow = tid >> 1, koct = (tid & 1) * 8;
  const GAS char* abase = (const GAS char*)resolve(d, g.A, g.mat) + (int64_t)(m0 + arow < M ? m0 + arow : M - 1) * g.sAm * 4;
  const int aslot = ((arow >> 5) * 2 + (tid & 1)) * 32 + (arow & 31);        // 16-byte unit inside a plane of the tile
  auto load_a = [&](u32x4 (&x)[4], int chunk) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = chunk * 32 + (v >> 1) * 16 + koct + (v & 1) * 4;
      const GAS u32x4* at = (const GAS u32x4*)(abase + (k < kend ? k : 0) * 4);
      if constexpr (ONCE) x[v] = __builtin_nontemporal_load(at);
      else x[v] = *at;
    }
  };
  auto stash_a = [&](u32x4& x, u32x4& y, int k, int buf) {                    // eight consecutive k of a row: one unit per plane
    asm volatile("" : "+v"(x), "+v"(y));          // nothing of this moves ahead of the step it stands in, where it would wait for the loads
    const bool okx = k < kend, oky = k + 4 < kend;                            // (K is a multiple of 4: whole vectors)
    uint32_t t0[3], t1[3], t2[3], t3[3];
    OperandBF<128, false, false, true>::split3(okx ? x.x : 0u, okx ? x.y : 0u, t0);
    OperandBF<128, false, false, true>::split3(okx ? x.z : 0u, okx ? x.w : 0u, t1);
    OperandBF<128, false, false, true>::split3(oky ? y.x : 0u, oky ? y.y : 0u, t2);
    OperandBF<128, false, false, true>::split3(oky ? y.z : 0u, oky ? y.w : 0u, t3);
#pragma unroll
    for (int c = 0; c < 3; ++c) lds_planes[(buf * SLOTS + 4 * c) * 64 + aslot] = u32x4{t0[c], t1[c], t2[c], t3[c]};
  };

  f32x16 acc[2][NBW];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int n = 0; n < NBW; ++n)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][n][i] = 0.f;
  auto compute = [&](int buf) {
    const u32x4* base = lds_planes + buf * SLOTS * 64 + lane;
    bf16x8 fa[3][2];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int a = 0; a < 2; ++a) fa[c][a] = __builtin_bit_cast(bf16x8, base[(4 * c + 2 * wm + a) * 64]);
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
      bf16x8 fb[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) fb[c] = __builtin_bit_cast(bf16x8, base[(ASLOTS + c * 2 * NBW + wn * NBW + n) * 64]);
#pragma unroll
      for (int ca = 0; ca < 3; ++ca)
#pragma unroll
        for (int cb = 0; cb + ca < 3; ++cb)
#pragma unroll
          for (int a = 0; a < 2; ++a) acc[a][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ca][a], fb[cb], acc[a][n], 0, 0, 0);
    }
  };

  u32x4 xa[4], xb[4];
  issue_b(0, 0);
  load_a(xa, 0);
  stash_a(xa[0], xa[1], koct, 0);
  WAIT_VM_BARRIER(0);
  for (int s = 0; s < nsteps; s += 2) {
    issue_b(s + 1, 1);
    load_a(xb, s / 2 + 1);                          // (past the end: element 0 of the row, replaced by zeros or not used)
    asm volatile("" ::: "memory");
    compute(0);
    stash_a(xa[2], xa[3], 16 * (s + 1) + koct, 1);
    WAIT_VM_BARRIER(4);
    issue_b(s + 2, 0);
    compute(1);
    stash_a(xb[0], xb[1], 16 * (s + 2) + koct, 0);
    WAIT_VM_BARRIER(0);
    xa[2] = xb[2];
    xa[3] = xb[3];
  }

  // accumulator register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32 of the block
  float* C = reinterpret_cast<float*>(const_cast<char*>(resolve(d, g.C, g.mat)));
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
      const int col = n0 + 32 * (wn * NBW + n) + (lane & 31);
      if (col >= N) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + 32 * (2 * wm + a) + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (row < M) *((GAS float*)C + (int64_t)row * g.ldc + col) = g.alpha * acc[a][n][v];
      }
    }
}

// B of the descriptors as three bf16 planes in operand layout (m = column n of B, k), zero outside K x N, at the
// matrix's place in three flat arrays.
__global__ __launch_bounds__(256) void k_pack_planes(DevCtx d, const GemmDesc* __restrict__ descs, uint16_t* __restrict__ p0,
                                                     uint16_t* __restrict__ p1, uint16_t* __restrict__ p2) {
  const GemmDesc g = descs[blockIdx.y];
  if (mat_skipped(d, g.mat)) return;
  const int64_t off = d.mats[g.mat].lr_off;
  const GAS float* B = (const GAS float*)resolve(d, g.B, g.mat);
  const int kgroups = (int)pad32(g.K) / 8, total = kgroups * (int)pad32(g.N);
  for (int i = (int)blockIdx.x * 256 + threadIdx.x; i < total; i += (int)gridDim.x * 256) {
    const int blk = i / (kgroups * 32), rem = i % (kgroups * 32);
    const int n = blk * 32 + (rem & 31), k = (rem >> 5) * 8;      // n fastest over the threads: a row of B is read contiguously
    uint32_t x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = n < g.N && k + e < g.K ? __float_as_uint(B[(int64_t)(k + e) * g.sBk + n * g.sBn]) : 0u;
    uint32_t t[4][3];
#pragma unroll
    for (int h = 0; h < 4; ++h) OperandBF<128, false, false, true>::split3(x[2 * h], x[2 * h + 1], t[h]);
    *((GAS u32x4*)(p0 + off) + i) = u32x4{t[0][0], t[1][0], t[2][0], t[3][0]};
    *((GAS u32x4*)(p1 + off) + i) = u32x4{t[0][1], t[1][1], t[2][1], t[3][1]};
    *((GAS u32x4*)(p2 + off) + i) = u32x4{t[0][2], t[1][2], t[2][2], t[3][2]};
  }
}

hipError_t launch_gemm_planes(const DevCtx& d, const GemmDesc* descs, int desc_first, int ndescs, const GemmTile* tiles, int ntiles, int tn_edge, bool a_once,
                              int64_t max_groups, uint16_t* p0, uint16_t* p1, uint16_t* p2, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const int64_t pack_blocks = (max_groups + 255) / 256;
  hipLaunchKernelGGL(k_pack_planes, dim3((unsigned)(pack_blocks < 1024 ? pack_blocks : 1024), ndescs), dim3(256), 0, s, d, descs + desc_first, p0, p1, p2);
  const dim3 grid((ntiles + 127) / 128 * 128), block(256);
#define LORDO_PLANES(NBWV, OV)                                                                                        \
  {                                                                                                                   \
    constexpr int LDS_BYTES = 2 * (12 + 6 * NBWV) * 1024;                                                             \
    static LdsRaised raised;                                                                                          \
    if (hipError_t e = raise_lds(reinterpret_cast<const void*>(k_gemm_planes<NBWV, OV>), LDS_BYTES, raised); e != hipSuccess) return e; \
    hipLaunchKernelGGL((k_gemm_planes<NBWV, OV>), grid, block, LDS_BYTES, s, d, descs, tiles, ntiles, p0, p1, p2);    \
  }
  if (tn_edge == 256) { if (a_once) LORDO_PLANES(4, true) else LORDO_PLANES(4, false) }
  else if (tn_edge == 128) { if (a_once) LORDO_PLANES(2, true) else LORDO_PLANES(2, false) }
  else if (tn_edge == 64) { if (a_once) LORDO_PLANES(1, true) else LORDO_PLANES(1, false) }
  else return hipErrorInvalidValue;
#undef LORDO_PLANES
  return hipGetLastError();
}

hipError_t launch_gemm32(const DevCtx& d, const GemmDesc* descs, const GemmTile* tiles, int ntiles, int tile, int mode, bool a_bf16,
                         hipStream_t s, float alpha_mul, int sub_m, int sub_n) {
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid(ntiles, sub_m, sub_n);
#define LORDO_GEMM(MODEV, BFV)                                                                                                        \
  {                                                                                                                                   \
    if (tile == 128) hipLaunchKernelGGL((k_gemm32<2, MODEV, BFV>), grid, dim3(256), 0, s, d, descs, tiles, a_bf16, alpha_mul, sub_m, sub_n); \
    else hipLaunchKernelGGL((k_gemm32<1, MODEV, BFV>), grid, dim3(256), 0, s, d, descs, tiles, a_bf16, alpha_mul, sub_m, sub_n);       \
  }
  if (mode == GEMM_ANY) LORDO_GEMM(GEMM_ANY, false)
  else if (mode == GEMM_RAGGED) { if (a_bf16) LORDO_GEMM(GEMM_RAGGED, true) else LORDO_GEMM(GEMM_RAGGED, false) }
  else { if (a_bf16) LORDO_GEMM(GEMM_ALIGNED, true) else LORDO_GEMM(GEMM_ALIGNED, false) }
#undef LORDO_GEMM
  return hipGetLastError();
}

}  // namespace lordo
