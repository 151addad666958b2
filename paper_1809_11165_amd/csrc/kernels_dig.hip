// Products with the block carried out on the 8-bit matrix pipe, to the accuracy of the fp64 one.
//
// V = K D needs fp32 kernel entries times an fp64 block, summed to fp64 accuracy (the CG recurrences
// amplify anything less).  On gfx950 the fp64 MFMA does that at 78.6 TFLOP/s and, running on the vector
// ALU, keeps every other vector instruction waiting.  The 8-bit MFMA (v_mfma_i32_16x16x64_i8: 16 cycles
// against 64 for v_mfma_f64_16x16x4) sums exactly in int32 and runs beside the vector ALU, so the same
// product is formed from digits:
//
//   entry   x = K kX, K <= 1, kX = 245 2^23, rounded to an integer: four balanced base-256 digits, which are
//           the four bytes of the word (x + 0x808080) ^ 0x808080;
//   block   D[i][q] 2^(62 - e_q) rounded to an integer, 2^e_q > max_i |D[i][q]|: eight balanced digits.
//
// The contraction index of ONE 16x16x64 MFMA is (16 rows) x (4 digits of the entry): the 16 x 16 tile of
// words, as the kernel function leaves it in the accumulator layout, IS the operand.  The other operand
// holds, for output pair (right-hand side q, weight w), the four digits w-3 .. w of D[i][q] (zero outside
// 0..7): digit a of the entry meets digit w - a of the block, so accumulator (q, w) collects every digit
// product of weight 256^-w, w = 0..7, exactly.  16 pairs share an MFMA: ceil(c / 2) of them per tile for
// c columns.  What is left out: three digit products of at most 2^14 at weight 8, so below 2^-60 of max|K| max|D| per
// term (2^e <= 2 max|D|, kX above 2^30), and D's rounding, 2^-62 max|D|.  Against a product of the same
// entries in extended precision the sums are as good as fp64 ones (1e-16 ... 2e-15 relative, fp64 accumulation
// 1e-16 ... 8e-16).  The entries are 32-bit numbers either way: in fixed point they are within 2.4e-10 of
// the largest or 2^-24 of themselves, whichever is more, where fp32 rounds them to 6e-8 of themselves: that suits dense
// blocks (see dig_dense).  What decides their error is their evaluation
// (3e-7), the rounding of the distance above all.  Product with normal columns, distance from the 64-bit
// result (this / k_mm_otf): 200,000 points, d = 8, 17 columns 5.3e-7 / 6.3e-7; 50,000, d = 16, 11 columns 3.3e-7 / 4.0e-7;
// 9,000, d = 4, 16 columns 1.76e-7 / 1.77e-7.
#include "bbmm_dig.h"
#include "bbmm_kfun.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short bf16x8u __attribute__((ext_vector_type(8)));

namespace {

// the same with k = 8 (lane/16) + element, fp32 sums
__device__ inline f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// kX k / s + kDigits, a whole number, from the scaled squared distance: the fp32 entry that unit_kernel gives, scaled.
// (The scale in the Matern coefficients would save the product, but overflow from distances of 1e15 on and round
// the coefficients once more.)
template <int KIND>
__device__ __forceinline__ float unit_kernel_x(float r2) {
  if (KIND == 0) return fmaf(__builtin_amdgcn_exp2f(-r2), kX, kRound);
  float a = __builtin_amdgcn_sqrtf(r2);
  float e = __builtin_amdgcn_exp2f(-a);
  return fmaf(fmaf(a, fmaf(a, kMatK2, kMatK1), 1.f) * e, kX, kRound);
}

// The digit words of a tile's four entries per lane in stages of a few vector instructions, so that the
// caller can place them between MFMAs.  v: -2 sgn x.x' on entry.  The norms are added as (|x|^2 + |x'|^2), never
// one after the other: entry (i, j) and entry (j, i) have to come out the same, bit for bit, or the iteration
// sees a matrix that is not symmetric (13 iterations more on 92 with the norms as the MFMA's addend).
template <int KIND>
struct DigEval {
  static constexpr int kStages = KIND == 0 ? 8 : 12;
  // constants of the evaluation, kept in scalar registers (as literals they double the size of most of the
  // instructions, and the loop is one long instruction stream)
  struct Const {
    int dig;
    float x, k1, k2;
    __device__ Const() : dig(kDigits), x(kX), k1(kMatK1), k2(kMatK2) {
      asm volatile("" : "+s"(dig), "+s"(x));
      if (KIND == 1) asm volatile("" : "+s"(k1), "+s"(k2));
    }
  };
  template <int S>
  static __device__ __forceinline__ void run(f32x4& v, f32x4& p, f32x4 sqi, float sqj, float sgn, i32x4& w, const Const& c) {
    constexpr int P = S >> 1, lo = 2 * (S & 1);                // half a tile per stage
    constexpr int E = KIND == 0 ? 2 : 4;                       // first stage of the conversion
#pragma unroll
    for (int r = lo; r < lo + 2; ++r) {
      if (KIND == 0) {
        if (P == 0) v[r] = __builtin_amdgcn_exp2f(-__builtin_fabsf(fmaf(v[r], sgn, sqi[r] + sqj)));
        if (P == 1) v[r] = fmaf(v[r], c.x, kRound);
      } else {
        if (P == 0) v[r] = __builtin_amdgcn_sqrtf(__builtin_fabsf(fmaf(v[r], sgn, sqi[r] + sqj)));
        if (P == 1) p[r] = __builtin_amdgcn_exp2f(-v[r]);
        if (P == 2) v[r] = fmaf(v[r], fmaf(v[r], c.k2, c.k1), 1.f);
        if (P == 3) v[r] = fmaf(v[r] * p[r], c.x, kRound);
      }
      if (P == E) w[r] = (int)v[r];
      if (P == E + 1) w[r] = w[r] ^ c.dig;
    }
  }
};

// Coordinates for the distance MFMA.  |x - x'|^2 = |x|^2 + |x'|^2 - 2 x.x'; the fp32 MFMA of the contraction
// runs on the vector ALU (measured: 14.4 ns a piece, added to the vector instructions around it), the
// bf16 one does not.  An fp32 coordinate is the sum of three bf16 pieces h + m + l exactly, and of the nine
// products all but l l' (2^-32) are kept: one v_mfma_f32_16x16x32_bf16 per four dimensions.
// The unit adds eight products (one lane group) at a time to the sum so far, so their order decides the error: the
// small ones of all dimensions first, m l' + l m', h l' + l h', h m' + m h', m m', and h h' last.  Rounding of
// 2 x.x', standard normal coordinates, d = 4, 8, 16: 1.5e-7, 1.7e-7, 2.7e-7 (fp32 MFMA 1.6e-7, 3.0e-7, 5.9e-7; all eight
// products of one dimension after those of another 2.1e-7, 3.6e-7, 6.5e-7).  A product and its mirror image are
// neighbours in one group, so that (i, j) and (j, i) get the same bits (see DigEval).  The unit aligns what it adds
// and drops bits downwards: -5e-8 to -7e-8 on average in the sums above, which would shift all entries
// the same way.  So every second block of 16 points enters with its sign turned: the sum of tile (I, J) is -2 x.x'
// times (-1)^(I + J), and the shift has either sign equally often.
__device__ inline unsigned short bf16_round(float v) {
  unsigned u = __float_as_uint(v);
  return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__device__ inline void bf16_pieces(float x, unsigned short (&q)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    q[k] = bf16_round(x);
    x -= __uint_as_float((unsigned)q[k] << 16);
  }
}

// Operand of lane group g, MFMA t, of one point: eight slots of the sum over (dimension, pair of pieces).  SIDE
// 0: the row's factors (times -2), 1: the column's.  x: the point's 4 KK coordinates, blk: its 16-row block.
template <int SIDE>
__device__ inline bf16x8u split_operand(const float* __restrict__ x, int KK, int blk, int t, int g) {
  int G = 4 * t + g, part = G / KK, u = G % KK;
  bf16x8u o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    unsigned short q[3];
    int k;
    if (part < 3) {                                // four dimensions, a product and its mirror image each
      bf16_pieces(x[4 * u + (e >> 1)], q);
      int a = part == 0 ? 1 : 0, b = part == 2 ? 1 : 2;      // m l, h l, h m
      k = ((e & 1) != SIDE) ? b : a;
    } else {                                       // m m of every dimension, then h h
      int s = 8 * u + e;
      k = s < 4 * KK ? 1 : 0;
      bf16_pieces(x[s < 4 * KK ? s : s - 4 * KK], q);
    }
    float v = __uint_as_float((unsigned)(k == 0 ? q[0] : (k == 1 ? q[1] : q[2])) << 16);
    if (SIDE == 0) v *= -2.f;
    o[e] = bf16_round(blk & 1 ? -v : v);           // (exact)
  }
  return o;
}

// column-side operand: Pb[i / 16][t][lane][8]
__global__ __launch_bounds__(256) void k_split_x(const float* __restrict__ Xs, int np, int KK, bf16x8u* __restrict__ Pb) {
  size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;      // MFMA operand order: [block][t][lane]
  if (idx >= (size_t)np * 4 * KK) return;
  int lane = (int)(idx & 63), t = (int)((idx >> 6) % KK);
  size_t row = (idx >> 6) / KK * 16 + (lane & 15);
  Pb[idx] = split_operand<1>(Xs + row * 4 * KK, KK, (int)(row >> 4), t, lane >> 4);
}

// One record per 16-row block holds everything a product needs of it, in 1 KB pieces of 16 bytes per lane
// (m = lane%16, g = lane/16): KK pieces of coordinates (row m, see split_operand), ng of digits, one of norms (rows 4g..4g+3).
// Digit piece p: for rows 4g..4g+3 the digit window of right-hand side 2 p + m/8, weight m%8.  One
// workgroup per record, first threads = (row quad, right-hand side).  Bound by the bytes written (128 per
// value).
__global__ __launch_bounds__(256) void k_digits(const double* __restrict__ D4, const float* __restrict__ Xs,
                                                 const float* __restrict__ sq, int n, int ld, int ng, int KK, int rec_bytes,
                                                 const DevState* __restrict__ st, unsigned* counts, char* __restrict__ rec) {
  if (st->done) return;
  int nrhs = 2 * ng;
  int rb = blockIdx.x;
  char* R = rec + (size_t)rb * rec_bytes;
  for (int e = threadIdx.x; e < KK * 64; e += 256)
    ((bf16x8u*)R)[e] = split_operand<0>(Xs + (size_t)(rb * 16 + (e & 15)) * 4 * KK, KK, rb, e >> 6, (e >> 4) & 3);
  if (KK > 0 && threadIdx.x < 64)
    ((f32x4*)(R + (KK + ng) * 1024))[threadIdx.x] = *(const f32x4*)(sq + rb * 16 + (threadIdx.x >> 4) * 4);
  if ((int)threadIdx.x >= 4 * nrhs) return;
  int g = threadIdx.x / nrhs, q = threadIdx.x % nrhs;
  unsigned hi = st->dmax[q];
  f64x4 d = *(const f64x4*)(D4 + ((size_t)(rb * 4 + g) * ld + q) * 4);
  int e = dig_exponent(hi);
  bool use = hi >= 0x00100000u && hi < 0x7ff00000u;   // neither zero nor non-finite
  unsigned long long str[4];
  unsigned small = 0, tiny = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    long long i = llrint(use ? ldexp(d[r], 62 - e) : 0.0);
    bool live = rb * 16 + 4 * g + r < n;
    small += live && llabs(i) < (1ll << 50);
    tiny += live && llabs(i) < (1ll << 42);
    constexpr long long C = 0x0080808080808080ll;
    str[r] = __builtin_bswap64((unsigned long long)((i + C) ^ C));   // most significant digit in byte 0
  }
  if (counts && small) {
    unsigned* c = counts + (rb % kDigCountRows) * 2 * BBMM_MAXC + q;
    atomicAdd(c, small);
    if (tiny) atomicAdd(c + BBMM_MAXC, tiny);
  }
  i32x4* out = (i32x4*)(R + (KK + (q >> 1)) * 1024) + g * 16 + (q & 1) * 8;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    i32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = (int)(unsigned)((str[r] << (8 * (7 - w))) >> 32);
    out[w] = v;
  }
}

// A workgroup's ring of records in LDS, shared by its four waves and copied straight from global memory (a
// wave copies every fourth piece; the last round may run past the record, hence whole multiples
// of 4 KB here, see bbmm_plan::dig_copy_offset).  In step k of a chunk record k - 1 feeds the digit MFMAs, k + 1 the distances, and
// k + kRing - 2 is requested, into the place that record k - 2 has left.
template <int KK, int NG>
struct DigRec {
  static constexpr int kPieces = bbmm_plan::dig_pieces(KK, NG);
  static constexpr int kBytes = bbmm_plan::dig_record_bytes(KK, NG);   // in global memory
  static constexpr int kCopies = bbmm_plan::dig_copies(KK, NG);        // per wave
  static constexpr int kSlot = bbmm_plan::dig_slot_bytes(KK, NG);      // in the ring
  static constexpr int kRing = bbmm_plan::dig_ring(KK, NG);
};

// Workgroup: 4 NJ column blocks (NJ per wave), a chunk of row blocks (an even number, at most
// kDigMaxBlocks: an accumulator grows by at most 2^20 per row block).  Partial sums of (K/s) D as
// k_mm_otf leaves them.
//
// In step k the wave evaluates the tiles of row block k on the vector ALU while the matrix pipe takes the
// digits of row block k - 1 and the distances of row block k + 1: all independent, so the two kinds are
// issued in turn.  The scheduler's own order and sched_group_barrier do not interleave them (the kinds
// then overlap a quarter of the time, whatever the number of waves): the order is written out, with a
// fence after every slot.  Operands come from LDS in batches of kB, requested one batch ahead, right after
// the first MFMA of the batch before (the wait there is for all of LDS).
//
// What bounds it: the vector ALU and the matrix pipe together.  Measured per SIMD with two waves: an 8-bit MFMA
// 7.8 ns, of which about 4 keep the vector ALU from issuing; a simple vector instruction 1.3 ns, a conversion
// 2.3 - 2.9, an exponential or square root 3.6.  A tile (16 x 16, 17 columns, RBF, d = 8) is 11 MFMAs and
// ~46 ns of vector work, one of Matern-5/2 with 11 columns at d = 16 is 10 and ~75 ns.
// Per product, n = 200 000, d = 8, 17 columns: 20.4 ms (k_mm_otf, fp64 matrix pipe: 32.1 ms); n = 32 000, d = 16,
// 11 columns, Matern-5/2: 0.62 ms (k_mm_otf_tri 0.82, k_mm_otf 0.99).
template <int KIND, int KK, int NG, int NJ>
__global__ __launch_bounds__(256, 2) void k_mm_otf_dig(const char* __restrict__ rec, const bf16x8u* __restrict__ Pb,
                                                        const float* __restrict__ sq, double* __restrict__ Vp, int np,
                                                        int ld, int nsplit, int blocks_per_split, int n,
                                                        const unsigned* __restrict__ counts, DevState* st) {
#ifdef __HIP_DEVICE_COMPILE__   // (the buffer resource type exists on the device only)
  if (counts) {                 // done is zero on entry and tells the kernels behind this one who did it
    if (!dig_dense(st, counts, n)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) st->done = 1;
  } else if (st->done) {
    return;
  }
  constexpr int LD = NG <= 8 ? 16 : 32;
  using Rec = DigRec<KK, NG>;
  constexpr int kRing = Rec::kRing;
  constexpr int kEpi = 4 * 16 * (LD + 1) * 8;
  __shared__ __align__(16) char lds[kRing * Rec::kSlot > kEpi ? kRing * Rec::kSlot : kEpi];
  int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int nblk = np >> 4;
  int split = blockIdx.x % nsplit, sstrip = blockIdx.x / nsplit;
  int jb0 = (sstrip * 4 + wave) * NJ;
  int jc = lane & 15, g = lane >> 4;
  int ib_begin = split * blocks_per_split;
  int ib_end = min(nblk, ib_begin + blocks_per_split);     // np is a multiple of 256: an even number of blocks
  if (ib_begin >= ib_end) {                                // (a last chunk may be empty: its slot is zero)
    for (int jb = 0; jb < NJ; ++jb)
      if (jb0 + jb < nblk)
        for (int q = g; q < LD; q += 4) Vp[((size_t)split * np + (size_t)((jb0 + jb) * 16 + jc)) * ld + q] = 0.0;
    return;
  }
  bf16x8 b[NJ][KK];
  float sqj[NJ];
  i32x4 acc[NJ][NG];
#pragma unroll
  for (int jb = 0; jb < NJ; ++jb) {
    int jblk = min(jb0 + jb, nblk - 1);      // (blocks beyond the matrix are computed and not stored)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) b[jb][kk] = __builtin_bit_cast(bf16x8, Pb[((size_t)jblk * KK + kk) * 64 + lane]);
    sqj[jb] = sq[jblk * 16 + jc];
#pragma unroll
    for (int q = 0; q < NG; ++q) acc[jb][q] = (i32x4){0, 0, 0, 0};
  }

  lds_char* L0 = (lds_char*)lds;
  int nk = ib_end - ib_begin;
  // the records as a raw buffer of this chunk (at most kDigMaxBlocks records of up to 21 KB and the room of
  // the last copy); past the end the last record comes again (the count of copies stays)
  __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(rec + (size_t)ib_begin * Rec::kBytes), 0,
                                                                  (int)bbmm_plan::dig_buffer_bytes(nk, KK, NG), 0x00020000);
  int voff = wave * 1024 + lane * 16;
  auto fetch = [&](int k, int slot) {
#pragma unroll
    for (int c = 0; c < Rec::kCopies; ++c)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(L0 + slot + wave * 1024 + c * 4096),
                                               16, voff, bbmm_plan::dig_copy_offset(KK, NG, k, nk, c), 0, 0);
  };
  // this lane's address in a ring place, opaque so that the constant offsets go into the instructions
  auto base = [&](int slot) {
    lds_char* q = L0 + slot + lane * 16;
    asm volatile("" : "+v"(q));
    return q;
  };
  auto next = [](int slot) { return slot + Rec::kSlot == kRing * Rec::kSlot ? 0 : slot + Rec::kSlot; };
  // (operands per batch: 16 kB registers; 17 and 18 columns fill the file otherwise, and the compiler then spills up to 48
  // registers inside the loop: n = 50 000, d = 8, 17 columns 1.65 ms, 1.30 without)
  constexpr int kOperands = NG + KK, kM = NJ * kOperands, kB = NG < 4 ? NG : (NG == 9 ? 3 : 4);
  constexpr int kS = NJ * DigEval<KIND>::kStages;
  typename DigEval<KIND>::Const cst;
  // sign of the sum of tile (k, jb): this times (-1)^(k + jb) (a chunk's first block is even)
  float sgn0 = __int_as_float(__builtin_amdgcn_readfirstlane(0x3f800000 | (int)((unsigned)jb0 << 31)));
  i32x4 op[2][kB];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 da[NJ], db[NJ], nrm;           // nrm: norms of block k's rows
  i32x4 wa[NJ], wb[NJ];
  // operand o of a step: digits of record k - 1 (address P), then coordinates of k + 1 (address Q)
  auto load_batch = [&](auto BB, lds_char* P, lds_char* Q) {
    constexpr int o0 = decltype(BB)::value * kB, o1 = o0 + kB < kOperands ? o0 + kB : kOperands;
    if constexpr (o0 < kOperands)
      static_for<o0, o1>([&](auto OO) {
        constexpr int o = decltype(OO)::value;
        op[(o / kB) & 1][o % kB] = *(lds_i32x4)(o < NG ? P + (KK + o) * 1024 : Q + (o - NG) * 1024);
      });
  };
  // slots of records k - 1, k, k + 1 and of the one requested in step k
  int s_prev = 0, s_cur = Rec::kSlot, s_next = 2 * Rec::kSlot, s_new = (kRing - 1) * Rec::kSlot;
  // d: distances of block k (used up), dn: of block k + 1; w: digits of block k - 1, wn: of block k
  auto step = [&](int k, auto odd, f32x4 (&d)[NJ], f32x4 (&dn)[NJ], const i32x4 (&w)[NJ], i32x4 (&wn)[NJ]) {
    wait_vm<(kRing - 4) * Rec::kCopies>();   // this wave's copies of record k + 1 have landed ...
    __builtin_amdgcn_s_barrier();            // ... and everybody's; nobody reads record k - 2 any more
    asm volatile("" ::: "memory");
    fetch(k + kRing - 2, s_new);
    lds_char* P = base(s_prev);
    lds_char* Q = base(s_next);
    f32x4 p;
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, kM>([&](auto MM) {
      constexpr int m = decltype(MM)::value, o = m / NJ, jb = m % NJ;
      const i32x4& a = op[(o / kB) & 1][o % kB];
      if constexpr (o < NG) acc[jb][o] = mfma_i8(a, w[jb], acc[jb][o]);
      else dn[jb] = mfma_bf16(__builtin_bit_cast(bf16x8, a), b[jb][o - NG], o == NG ? zero : dn[jb]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (jb == 0 && o % kB == 0) {
        load_batch(std::integral_constant<int, o / kB + 1>{}, P, Q);
      }
      static_for<m * kS / kM, (m + 1) * kS / kM>([&](auto SS) {
        constexpr int S = decltype(SS)::value, t = S / DigEval<KIND>::kStages;
        DigEval<KIND>::template run<S % DigEval<KIND>::kStages>(d[t], p, nrm, sqj[t], (decltype(odd)::value + t) & 1 ? -sgn0 : sgn0,
                                                                wn[t], cst);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    load_batch(std::integral_constant<int, 0>{}, base(s_cur), Q);    // first operands of the next step
    nrm = *(lds_f32x4)(Q + (Rec::kPieces - 1) * 1024);
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) asm volatile("" : "+v"(wn[jb]), "+v"(dn[jb]));   // done here, not where used
    s_prev = s_cur;
    s_cur = s_next;
    s_next = next(s_next);
    s_new = next(s_new);
  };
  // blocks 0 and 1: distances, tiles of block 0
#pragma unroll
  for (int k = 0; k < kRing - 1; ++k) fetch(k, k * Rec::kSlot);
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  {
    f32x4 p;
    lds_char *P = base(0), *Q = base(Rec::kSlot);
    nrm = *(lds_f32x4)(P + (Rec::kPieces - 1) * 1024);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      bf16x8 a0 = __builtin_bit_cast(bf16x8, *(lds_i32x4)(P + kk * 1024));
      bf16x8 a1 = __builtin_bit_cast(bf16x8, *(lds_i32x4)(Q + kk * 1024));
#pragma unroll
      for (int jb = 0; jb < NJ; ++jb) {
        db[jb] = mfma_bf16(a0, b[jb][kk], kk == 0 ? zero : db[jb]);
        da[jb] = mfma_bf16(a1, b[jb][kk], kk == 0 ? zero : da[jb]);
      }
    }
    static_for<0, kS>([&](auto SS) {
      constexpr int S = decltype(SS)::value, t = S / DigEval<KIND>::kStages;
      DigEval<KIND>::template run<S % DigEval<KIND>::kStages>(db[t], p, nrm, sqj[t], t & 1 ? -sgn0 : sgn0, wa[t], cst);
    });
    load_batch(std::integral_constant<int, 0>{}, P, P);
    nrm = *(lds_f32x4)(Q + (Rec::kPieces - 1) * 1024);
  }
#pragma unroll 1
  for (int k = 1; k + 1 < nk; k += 2) {
    step(k, std::integral_constant<int, 1>{}, da, db, wa, wb);
    step(k + 1, std::integral_constant<int, 0>{}, db, da, wb, wa);
  }
  step(nk - 1, std::integral_constant<int, 1>{}, da, db, wa, wb);
  {
    lds_char* P = base(s_prev);
    static_for<0, NJ * NG>([&](auto MM) {
      constexpr int m = decltype(MM)::value, q = m / NJ, jb = m % NJ;
      i32x4 a = *(lds_i32x4)(P + (KK + q) * 1024);
      acc[jb][q] = mfma_i8(a, wb[jb], acc[jb][q]);
    });
  }
  wait_vm<0>();                              // copies nobody waited for
  // The diagonal has distance zero exactly, the expansion gives a rounding error: the difference of its
  // entries, kX less what the loop used (the same instructions give the same bits), is added here, once per
  // column block, instead of testing for it in every tile.
#pragma unroll
  for (int jb = 0; jb < NJ; ++jb) {
    int ib = jb0 + jb;
    if (ib >= ib_begin && ib < ib_end) {
      const i32x4* R = (const i32x4*)(rec + (size_t)ib * Rec::kBytes) + lane;
      f32x4 sqi = *(const f32x4*)(sq + ib * 16 + g * 4), d2 = zero;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) d2 = mfma_bf16(__builtin_bit_cast(bf16x8, R[kk * 64]), b[jb][kk], d2);
      i32x4 w;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int x = (int)unit_kernel_x<KIND>(__builtin_fabsf(d2[r] + (sqi[r] + sqj[jb])));   // (the sign is (-1)^(2 I) here)
        w[r] = 4 * g + r == jc ? (((int)kX + kDigits - x + kDigits) ^ kDigits) : 0;
      }
#pragma unroll
      for (int q = 0; q < NG; ++q) acc[jb][q] = mfma_i8(R[(KK + q) * 64], w, acc[jb][q]);
    }
  }
  __syncthreads();
  double* T = (double*)lds + wave * (16 * (LD + 1));
  double* vout = Vp + (size_t)split * np * ld;
#pragma unroll
  for (int jb = 0; jb < NJ; ++jb)
    if (jb0 + jb < nblk)
      dig_store<NG, LD>(acc[jb], 1.0 / (double)kX, T, jc, g, st, vout + (size_t)((jb0 + jb) * 16 + jc) * ld);
#endif
}

}  // namespace

// Column pairs per product, rounded up to a compiled count.  A pair is one MFMA more per tile; n = 20 000, d = 8, RBF, 4,
// 8, 12, 16, 18, 24, 32 columns: 155, 172, 202, 226, 258, 310, 385 us.
int dig_groups(int c) {
  for (int g : {2, 4, 6, 8, 9, 12, 16})
    if (c <= 2 * g) return g;
  return 16;
}

void launch_digits(hipStream_t s, const double* D4, const float* Xs, const float* sq, int n, int np, int ld, int KK, int ng,
                   const DevState* st, unsigned* counts, void* rec) {
  k_digits<<<np / 16, 256, 0, s>>>(D4, Xs, sq, n, ld, ng, KK, bbmm_plan::dig_record_bytes(KK, ng), st, counts, (char*)rec);
}

// Column blocks per wave: what the accumulators (4 ng registers a block), the coordinates (4 KK) and the tiles in flight
// (24) leave room for in the 256 registers that two waves per SIMD have, without spills inside the loop
// (n = 50 000, d = 16, 11 columns: 1433 us with 4, 1597 with 3; n = 100 000, d = 8, 17 columns: 5272 with 4, 5632 with 3).
// The widest records (9 to 16 dimensions, 25 to 32 columns) leave LDS for one workgroup and so one wave per SIMD.
int dig_nj(int KK, int ng) {
  if (ng == 2) return KK <= 2 ? 6 : 5;
  if (ng == 4) return KK <= 2 ? 5 : 4;
  if (ng == 6) return 4;
  if (ng <= 9) return KK <= 2 ? 4 : 3;
  return ng == 12 && KK <= 2 ? 3 : 2;
}

void launch_split_x(hipStream_t s, const float* Xs, int np, int KK, void* Pb) {
  size_t total = (size_t)np * 4 * KK;
  k_split_x<<<(int)((total + 255) / 256), 256, 0, s>>>(Xs, np, KK, (bf16x8u*)Pb);
}

int launch_mm_otf_dig(hipStream_t s, int kernel, int KK, int ng, const void* rec, const void* Pb, const float* sq,
                      double* Vp, int n, int np, int ld, int nsplit, const unsigned* counts, DevState* st) {
  int nblk = np / 16;
  int bps = (nblk + nsplit - 1) / nsplit;
  bps += bps & 1;
  if (bps > kDigMaxBlocks) return 1;
  int nj = dig_nj(KK, ng);
  int grid = ((nblk + 4 * nj - 1) / (4 * nj)) * nsplit;
#define DIG(K, G, J)                                                                                           \
  if (kernel == 0)                                                                                             \
    k_mm_otf_dig<0, K, G, J><<<grid, 256, 0, s>>>((const char*)rec, (const bf16x8u*)Pb, sq, Vp, np, ld, nsplit, bps, n, counts, st); \
  else                                                                                                         \
    k_mm_otf_dig<1, K, G, J><<<grid, 256, 0, s>>>((const char*)rec, (const bf16x8u*)Pb, sq, Vp, np, ld, nsplit, bps, n, counts, st)
#define DIG_G(K, TWO, FOUR, NINE, TWELVE)  \
  switch (ng) {                            \
    case 2: DIG(K, 2, TWO); break;         \
    case 4: DIG(K, 4, FOUR); break;        \
    case 6: DIG(K, 6, 4); break;           \
    case 8: DIG(K, 8, NINE); break;        \
    case 9: DIG(K, 9, NINE); break;        \
    case 12: DIG(K, 12, TWELVE); break;    \
    case 16: DIG(K, 16, 2); break;         \
    default: return 1;                     \
  }
  switch (KK) {   // column blocks per wave as dig_nj says
    case 1: DIG_G(1, 6, 5, 4, 3); break;
    case 2: DIG_G(2, 6, 5, 4, 3); break;
    case 4: DIG_G(4, 5, 4, 3, 2); break;
    default: return 1;   // beyond 16 dimensions the coordinates (4 KK registers a block) leave too few blocks a wave
  }
#undef DIG_G
#undef DIG
  return 0;
}
