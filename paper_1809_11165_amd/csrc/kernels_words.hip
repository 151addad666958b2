// K_hat kept as digit words: the matrix of an iteration whose products run on the 8-bit matrix pipe (gfx950 / CDNA4).
//
// The triangle product on the fp64 matrix pipe (k_mm_sym) is bound by that pipe and by the vector instructions it
// blocks: 1.28 ms at n = 50 000, 11 columns, where reading the triangle takes 0.73 ms.  Digits (see kernels_dig.hip) need
// a quarter of the matrix time; turning stored fp32 entries into digit words inside the product, though, costs three vector
// instructions and two LDS passes per entry and leaves 1.35 ms (measured).  So the words themselves are stored, which takes
// 1.08 ms (n = 20 000: 0.19 ms, whole fp32 matrix 0.25): K / s
// as 31-bit fixed point, four balanced base-256 digits in four bytes, laid out as the product reads them.
//
// Layout: panels of BBMM_WORDS_PANEL columns, panel P keeping rows [0, (P + 1) * BBMM_WORDS_PANEL) (the upper triangle, blocks
// on the diagonal whole); 16-row steps of 32 tiles, a tile (16 x 16) being 1 KB: rows 4 a .. 4 a + 3 of column c are the 16
// bytes in place (c ^ a) of the tile's a-th 256 bytes.  For blocks of more than 16 columns (k_mm_words_wide) every panel keeps all
// rows ("whole").  A column quadruple is then one 16-byte read per lane, and
// a row's four words of a column quadruple four 4-byte reads, both without bank conflicts.  The diagonal is zero here and
// added afterwards (addD), which keeps it exact.
#include "bbmm_dig.h"
#include "bbmm_kfun.h"

namespace {

constexpr int kWP = BBMM_WORDS_PANEL;
constexpr int kWTiles = kWP / 16;                            // tiles per 16-row step

// first step of panel P (whole: of np rows each)
__host__ __device__ inline size_t words_panel_step(int P) { return (size_t)(kWP / 16) * ((size_t)P * (P + 1) / 2); }
__host__ __device__ inline size_t words_panel_step(int P, int np, int whole) { return whole ? (size_t)(np / 16) * P : words_panel_step(P); }

__device__ inline f64x4 mfma16d(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Centred, scaled inputs in fp64: Xo[(b * KK + kk) * 64 + l] = xs[16 b + l%16][4 kk + l/16] (zero for padding), sqo[i] = |xs_i|^2.
__global__ __launch_bounds__(256) void k_prep_words(const float* __restrict__ X, int n, int d, int np, int KK, HypArgs hyp,
                                                     const DevState* __restrict__ st, double* __restrict__ Xo, double* __restrict__ sqo) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= np) return;
  double s = 0.0;
  for (int dim = 0; dim < 4 * KK; ++dim) {
    double v = (i < n && dim < d) ? ((double)X[(size_t)i * d + dim] - st->xmean[dim]) * hyp.xscale[dim] : 0.0;
    Xo[((size_t)(i >> 4) * KK + (dim >> 2)) * 64 + (dim & 3) * 16 + (i & 15)] = v;
    s = fma(v, v, s);
  }
  sqo[i] = s;
}

// k / s as a digit word: rounded to the fixed-point grid once (fp32 arithmetic would round entries above 2^-8 once more).
__device__ inline int entry_word(double k) { return ((int)rint(k * (double)kX) + kDigits) ^ kDigits; }

// One wave: the tiles of one 16-row step of a panel, in turn.  Distances by fp64 MFMA (rows in the order 4 (m % 4) + m / 4, so
// that a lane's four results are four consecutive rows), the kernel function in fp32.  Bound by the stores.
// An entry that is no number (a squared distance beyond fp32: Matern, infinity times zero) has no word: it sets st->xbad, on which the
// products return NaN and the run is made again with the fp32 entries.
template <int KIND>
__global__ __launch_bounds__(256) void k_build_words(const double* __restrict__ Xo, const double* __restrict__ sqo, int n, int np,
                                                      int KK, int whole, DevState* __restrict__ st, int* __restrict__ Kw) {
  int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int jc = lane & 15, g = lane >> 4;
  int P = blockIdx.x, step = blockIdx.y * 4 + wave;
  if (step * 16 >= (whole ? np : min(np, (P + 1) * kWP))) return;
  const double* Ar = Xo + (size_t)step * KK * 64 + g * 16 + 4 * (jc & 3) + (jc >> 2);
  double si[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) si[r] = sqo[step * 16 + 4 * g + r];
  int ntiles = min(kWTiles, (np - P * kWP) / 16);
  int* out = Kw + ((words_panel_step(P, np, whole) + step) * kWTiles) * 256 + (g * 16 + (jc ^ g)) * 4;
  bool bad = false;
  for (int t = 0; t < ntiles; ++t) {
    int cb = P * kWTiles + t;
    const double* Br = Xo + (size_t)cb * KK * 64 + lane;
    double sj = sqo[cb * 16 + jc];
    f64x4 acc;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = si[r] + sj;
    for (int kk = 0; kk < KK; ++kk) acc = mfma16d(-2.0 * Ar[kk * 64], Br[kk * 64], acc);
    i32x4 w;
    int j = cb * 16 + jc;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int i = step * 16 + 4 * g + r;
      float r2 = __builtin_fabsf((float)acc[r]);
      float k = unit_kernel<KIND>(r2);
      bool entry = i != j && i < n && j < n;
      bad |= entry && !(k == k);
      w[r] = entry ? entry_word((double)fminf(k, 1.f)) : 0;
    }
    __builtin_nontemporal_store(w, (i32x4*)(out + (size_t)t * 256));
  }
  if (bad) st->xbad = 1;
}

// The same from a stored fp32 matrix (layout as for launch_copy_block), whose entries are s K: an iteration started on a matrix
// that its caller has had built runs on the entries of that matrix.  (No word: NaN as above, and infinity, of an outputscale beyond fp32.)
__global__ __launch_bounds__(256) void k_words_of(const float* __restrict__ K, size_t pw, int tri, double inv_s, int n, int np,
                                                   int whole, DevState* __restrict__ st, int* __restrict__ Kw) {
  int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int jc = lane & 15, g = lane >> 4;
  int P = blockIdx.x, step = blockIdx.y * 4 + wave;
  if (step * 16 >= (whole ? np : min(np, (P + 1) * kWP))) return;
  int ntiles = min(kWTiles, (np - P * kWP) / 16);
  int* out = Kw + ((words_panel_step(P, np, whole) + step) * kWTiles) * 256 + (g * 16 + (jc ^ g)) * 4;
  bool bad = false;
  for (int t = 0; t < ntiles; ++t) {
    int j = (P * kWTiles + t) * 16 + jc;
    size_t q = (size_t)j / pw;                               // (the panels of a triangle are 1 024 wide: rows up to this step are there)
    const float* src = K + (tri ? pw * pw * (q * (q + 1) / 2) : q * (size_t)np * pw) + (size_t)j % pw;
    i32x4 w;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int i = step * 16 + 4 * g + r;
      float v = src[(size_t)i * pw];
      bool entry = i != j && i < n && j < n;
      bad |= entry && !(v < __builtin_inff());
      w[r] = entry ? entry_word(fmin((double)v * inv_s, 1.0)) : 0;
    }
    __builtin_nontemporal_store(w, (i32x4*)(out + (size_t)t * 256));
  }
  if (bad) st->xbad = 1;
}

// Geometry of the product for blocks of up to 2 NG columns: a wave owns 128 matrix columns, a workgroup of four waves one panel.
template <int NG>
struct WordsMM {
  static constexpr int kNJ = 8;                              // 16-column tiles per wave
  static constexpr int kSlotK = 4 * kNJ * 1024;              // a 16-row step of the matrix, all waves
  static constexpr int kRounds = (NG + 3) / 4;               // a step's digit record, copied four pieces at a time
  static constexpr int kSlotD = NG * 1024;
  static constexpr int kRingK = 4, kRingD = 3;
  static constexpr int kSP = 2 * NG + 1;                     // doubles per staged row of the row side
  static constexpr int kStage = 4 * 16 * kSP * 8;            // all waves
  static constexpr int kOffD = kRingK * kSlotK;
  static constexpr int kOffS = kOffD + kRingD * kSlotD;
  static constexpr int kLds = kOffS + 2 * kStage;
  // copies that a wave has requested behind record k + 1 when step k waits for it: those of a step from there to the same place of
  // the next (kNJ + kRounds), and the tiles of that one up to the wait (kNJ - 1)
  static constexpr int kAhead = 2 * kNJ + kRounds - 1;
  static_assert(kLds <= 160 * 1024 && NG % 2 == 0, "");
};

// out[J] += T^T D[I] and out[I] += T D[J] for every tile T above the diagonal blocks; inside them (stored whole) the first only
// (the second is formed and dropped: they are one step in (P + 1), and a loop of its own costs more than it saves).
// Work list: runs of rows of a panel (MmPiece), dealt out in equal shares; a piece's column sums go to its slot of the panel's
// rows, the row sums of panel P for output rows of panel s < P to slot slot_base[s] + P - s - 1.  A workgroup walks down the
// rows of a piece; column sums (acc) and the columns' digits (dj) stay in registers for the whole of it, the rows' digits (op)
// and sums (ra) for a step.  Matrix and records are copied straight into LDS, three steps ahead; a step has one barrier.
template <int NG>
__global__ __launch_bounds__(256, 1) void k_mm_words(const int* __restrict__ Kw, const char* __restrict__ rec, double* __restrict__ Vp,
                                                     int np, int ld, const MmPiece* __restrict__ pieces, const int* __restrict__ first,
                                                     const int* __restrict__ slot_base, const DevState* __restrict__ st) {
#ifdef __HIP_DEVICE_COMPILE__   // (the buffer resource type exists on the device only)
  if (st->done) return;
  using G = WordsMM<NG>;
  constexpr int NJ = G::kNJ;
  static_assert(kWTiles == 4 * NJ, "a workgroup covers one panel");
  __shared__ __align__(1024) char lds[G::kLds];
  lds_char* L0 = (lds_char*)lds;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jc = lane & 15, g = lane >> 4;
  // this lane's places in a tile: column jc, rows 4 g ..; row jc, columns 4 g + r
  const int colp = (g * 16 + (jc ^ g)) * 16;
  int rowp[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) rowp[r] = (jc >> 2) * 256 + ((4 * g + r) ^ (jc >> 2)) * 16 + (jc & 3) * 4;
  const int ks0 = wave * (NJ * 1024);
  double* const S = (double*)(lds + G::kOffS);               // staged row sums: [wave][step parity][row][kSP]
  const i32x4 zero4 = {0, 0, 0, 0};
  // weights of a lane's four accumulators: 2^16 and 1, or 2^-32 times that (weights 4 .. 7)
  const double wlo = (g & 1) ? 0x1p-32 : 1.0, whi = 65536.0 * wlo;
  // Way out of the sums, for one block column per thread: position fpos of an output row is column fcol.  (Digits of a zero or
  // non-finite column are zero.)
  const int frow = threadIdx.x >> 4, fpos = threadIdx.x & 15, fcol = 4 * (fpos & 3) + (fpos >> 2);
  const bool fuse = fcol < 2 * NG;
  const int fv = frow * G::kSP + min(fcol, 2 * NG - 1), fst = frow * ld + fpos;
  const unsigned fhi = fuse ? st->dmax[fcol] : 0u;
  const int fex = dig_exponent(fhi) + 18 - 24;
  const double fspec = fuse ? dig_special(fhi, st->dflag[fcol], st->xbad) : 0.0;
  const double fscale = fuse ? 1.0 / (double)kX : 0.0;

  i32x4 acc[NJ][NG], dj[NJ][NG], op[NG], ra[NG], wc[2], wr[2];

  const int pb = first[blockIdx.x], pe = first[blockIdx.x + 1];
  MmPiece P = pieces[pb];
  int nk, colw;
  bool active;
  const int* kb;
  const char* db;
  auto fetch_k1 = [&](int k, int slot, int e) {
    __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)kb, 0, ((nk - 1) * kWTiles + NJ) * 1024, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (__attribute__((address_space(3))) void*)(L0 + slot + ks0 + e * 1024), 16, lane * 16,
                                             k * (kWTiles * 1024) + e * 1024, 0, 2);
  };
  auto fetch_d = [&](int k, int slot) {    // (a round's pieces past the record are its last again)
    __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)db, 0, nk * NG * 1024, 0x00020000);
#pragma unroll
    for (int c = 0; c < G::kRounds; ++c) {
      int piece = min(c * 4 + wave, NG - 1);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rd, (__attribute__((address_space(3))) void*)(L0 + G::kOffD + slot + piece * 1024), 16,
                                               lane * 16, k * (NG * 1024) + piece * 1024, 0, 0);
    }
  };
  // what a piece needs before its first step: its first steps and records, its columns' digits
  auto open_piece = [&]() {
    nk = (P.row_end - P.row_begin) >> 4;   // (1 .. kDigMaxBlocks)
    colw = P.strip * kWP + wave * (16 * NJ);
    active = colw < np;                    // np is a multiple of 256: all of a wave's columns or none
    kb = Kw + ((words_panel_step(P.strip) + (P.row_begin >> 4)) * kWTiles + wave * NJ) * 256;
    db = rec + (size_t)(P.row_begin >> 4) * (NG * 1024);
#pragma unroll
    for (int k = 0; k < G::kRingK; ++k) {
      if (k < G::kRingD && k < nk) fetch_d(k, k * G::kSlotD);
      if (active && k < nk)
#pragma unroll
        for (int e = 0; e < NJ; ++e) fetch_k1(k, k * G::kSlotK, e);
    }
    if (active)
#pragma unroll
      for (int b = 0; b < NJ; ++b)
#pragma unroll
        for (int q = 0; q < NG; ++q) dj[b][q] = *(const i32x4*)(rec + ((size_t)(colw / 16 + b) * NG + q) * 1024 + lane * 16);
  };
  open_piece();

#pragma unroll 1
  for (int pi = pb; pi < pe; ++pi) {
#pragma unroll
    for (int b = 0; b < NJ; ++b)
#pragma unroll
      for (int q = 0; q < NG; ++q) acc[b][q] = zero4;
#pragma unroll
    for (int q = 0; q < NG; ++q) ra[q] = zero4;
    if (!active)                           // no sums of its own in this piece
      for (int i = lane; i < 2 * 16 * G::kSP; i += 64) S[wave * 2 * 16 * G::kSP + i] = 0.0;
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    double f = 0.0, fn = 0.0;
    double* vslot = Vp;
    auto part = [&](int i, int k) { return S[(i * 2 + (k & 1)) * 16 * G::kSP + fv]; };   // wave i's
    auto flush = [&](auto II, int k) {     // stages 0..3: add one wave's part (fn); 4, 5: scale; 6: store
      constexpr int i = decltype(II)::value;
      if constexpr (i < 4) f = i == 0 ? fn : f + fn;
      if constexpr (i == 4) f *= fscale;
      if constexpr (i == 5) f = ldexp(f, fex) + fspec;
      if constexpr (i == 6) {
        int row0 = P.row_begin + 16 * k;
        if (row0 < P.strip * kWP) {
          if (k == 0 || row0 % kWP == 0) {                   // a new panel of rows
            int so = row0 / kWP;
            vslot = Vp + (size_t)(slot_base[so] + (P.strip - so - 1)) * np * ld;
          }
          (vslot + (size_t)row0 * ld)[fst] = f;
        }
      }
    };
    auto flush_all = [&](int k) {
      static_for<0, 7>([&](auto II) {
        if constexpr (decltype(II)::value < 4) fn = part(decltype(II)::value, k);
        flush(II, k);
      });
    };
    // Four accumulators per piece and lane to doubles in LDS, two pieces (four block columns) in five stages: lanes g, g ^ 1 hold the
    // two halves of the weights.  (An entry's top digit is at most 123, its others at most 128, as are the block's: 128 terms of 128 (123 + 3 * 128) in a step,
    // 8.31e6, times 257: 2.135e9 < 2^31.)
    int sh[2], sl[2];
    double sx[2];
    constexpr int kStages = 5 * (NG / 2), kEarly = NG >= 4 ? NG / 2 : 0;     // of these, the first in the last instructions of the step itself
    double* const sw = S + (wave * 32 + jc) * G::kSP + 2 * (g & 1) + (g >> 1);
    auto stage = [&](auto II, int k) {
      constexpr int i = decltype(II)::value % 5, e = 2 * (decltype(II)::value / 5);
      if constexpr (i == 0) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          sh[c] = (ra[e + c][0] << 8) + ra[e + c][1];
          sl[c] = (ra[e + c][2] << 8) + ra[e + c][3];
        }
      }
      if constexpr (i == 1) {
        sx[0] = (double)sl[0] * wlo;
        sx[1] = (double)sl[1];
      }
      if constexpr (i == 2) sx[1] *= wlo;
      if constexpr (i == 3) {
#pragma unroll
        for (int c = 0; c < 2; ++c) sx[c] = fma((double)sh[c], whi, sx[c]);
      }
      if constexpr (i == 4) {
        // rows of 16 lanes g = 0..3: x0 = [a0 a1 a2 a3], x1 = [b0 b1 b2 b3] -> [a0 b0 a2 b2] + [a1 b1 a3 b3]
        auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(sx[0]), (unsigned)__double2loint(sx[1]), false, false);
        auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(sx[0]), (unsigned)__double2hiint(sx[1]), false, false);
        sw[(k & 1) * 16 * G::kSP + 2 * e] = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
      }
    };
    // ring places of a step: k0 of step k, k1 of step k + 1, d0 and d1 of their records; what step k frees is k0 and d0
    int k0 = 0, k1 = G::kSlotK, kf = 0, d0 = 0, d1 = G::kSlotD;   // kf: of step k - 1
    lds_char* const pd = L0 + G::kOffD + lane * 16;
    auto rd_col = [&](int p, int b) { return *(lds_i32x4)(L0 + p + colp + b * 1024); };
    auto rd_row = [&](int p, int b, int e) { return *(const __attribute__((address_space(3))) int*)(L0 + p + rowp[e] + b * 1024); };
    if (active) {
#pragma unroll
      for (int q = 0; q < NG; ++q) op[q] = *(lds_i32x4)(pd + q * 1024);
      wc[0] = rd_col(k0 + ks0, 0);
      wc[1] = rd_col(k0 + ks0, 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) wr[0][e] = rd_row(k0 + ks0, 0, e);
    }
    // Tiles two at a time, in 4 NG matrix instructions: columns of both, then rows of both.  Whatever else a step does is dealt
    // out behind single matrix instructions, up to three vector instructions each (one wave per SIMD: nothing else fills the
    // time; measured, ns per matrix instruction with 0 .. 4 vector instructions behind it: 7.7, 8.9, 9.5, 9.8, 12.7).
    // A tile's words are requested where the last but one's registers become free, 3 NG instructions ahead of their use.
#pragma unroll 1
    for (int k = 0; k < nk; ++k) {
      if (active) {
        static_for<0, NJ / 2>([&](auto PP) {
          constexpr int p = decltype(PP)::value, bn = p == NJ / 2 - 1 ? 0 : 2 * p + 2;
          if constexpr (p == NJ / 2 - 1) {
            if (k + G::kRingK >= nk) wait_vm<0>();
            else wait_vm<G::kAhead>();                       // (row sums stored since are not counted: inside the diagonal block there are none)
            // This wave's copies of step k + 1 and record k + 1 have landed, and so, behind the barrier, have everybody's.  So
            // have the row sums of step k - 1 (LDS works in order, and words read behind them have been used).
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
          }
          const int kn = (p == NJ / 2 - 1 ? k1 : k0) + ks0;
          static_for<0, 4 * NG>([&](auto MM) {
            constexpr int m = decltype(MM)::value, ph = m / NG, q = m % NG, b = 2 * p + (ph & 1);
            if constexpr (ph < 2) acc[b][q] = mfma_i8(op[q], wc[ph], acc[b][q]);
            else ra[q] = mfma_i8(dj[b][q], wr[ph & 1], b == 0 ? zero4 : ra[q]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (m < 4) wr[1][m] = rd_row(k0 + ks0, 2 * p + 1, m);
            if constexpr (m == NG) wc[0] = rd_col(kn, bn);
            if constexpr (m == 2 * NG) wc[1] = rd_col(kn, bn + 1);
            if constexpr (ph == 3)
              static_for<q * 4 / NG, (q + 1) * 4 / NG>([&](auto EE) { wr[0][decltype(EE)::value] = rd_row(kn, bn, decltype(EE)::value); });
            // places of the two tiles before this pair receive those of four steps on (a copy at a time: the address unit takes one
            // from each of the four waves in 64 cycles)
            if constexpr (m == NG - 1 || m == 3 * NG - 1) {
              constexpr int t = (2 * p + NJ - 2 + (m > NG)) % NJ;
              if (p == 0 ? k > 0 && k + G::kRingK - 1 < nk : k + G::kRingK < nk)
                fetch_k1(p == 0 ? k + G::kRingK - 1 : k + G::kRingK, p == 0 ? kf : k0, t);
            }
            if constexpr (p == 0 && ph < 2)                  // (row sums of the step before: the row side starts over behind this)
              static_for<kEarly + m * (kStages - kEarly) / (2 * NG), kEarly + (m + 1) * (kStages - kEarly) / (2 * NG)>(
                  [&](auto II) { stage(II, k - 1); });       // (of no step before the first; not used then)
            if constexpr (p == 1 && m % NG == 0) fn = part(ph, k - 2);       // (of no step before the third; not used then)
            if constexpr (p == 1 && m % NG == NG - 1) flush(std::integral_constant<int, ph>{}, k - 2);
            if constexpr (p == 2 && m % NG == 0) {
              if constexpr (ph < 2) flush(std::integral_constant<int, 4 + ph>{}, k - 2);
              if constexpr (ph == 2) {
                if (k > 1) flush(std::integral_constant<int, 6>{}, k - 2);
              }
            }
            if constexpr (p == NJ / 2 - 1) {
              if constexpr (4 * NG - 1 - m < kEarly) stage(std::integral_constant<int, kEarly - (4 * NG - m)>{}, k);
              if constexpr (ph == 1) op[q] = *(lds_i32x4)(pd + d1 + q * 1024);
              if constexpr (ph == 2 && q == 0) {
                if (k + G::kRingD < nk) fetch_d(k + G::kRingD, d0);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          });
        });
      } else {
        if (k > 1) flush_all(k - 2);
        wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (k + G::kRingD < nk) fetch_d(k + G::kRingD, d0);
      }
      kf = k0;
      k0 = k1;
      k1 = k1 + G::kSlotK == G::kRingK * G::kSlotK ? 0 : k1 + G::kSlotK;
      d0 = d1;
      d1 = d1 + G::kSlotD == G::kRingD * G::kSlotD ? 0 : d1 + G::kSlotD;
    }
    if (active) static_for<0, kStages>([&](auto II) { stage(II, nk - 1); });
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (nk > 1) flush_all(nk - 2);
    flush_all(nk - 1);
    // the next piece's first copies travel while this one's column sums are stored (a wave's rows of S for its own use)
    const bool store = active;
    double* vout = Vp + ((size_t)P.slot * np + colw) * ld;
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (pi + 1 < pe) {
      P = pieces[pi + 1];
      open_piece();
    }
    if (store) {
      double* T = S + wave * 2 * 16 * G::kSP;
      int frw = lane >> 4;                 // (opaque: the compiler would form and spill all addresses before the main loop)
      asm volatile("" : "+v"(frw));
      const int voff = (frw * ld + fpos) * 8;
      static_for<0, NJ>([&](auto BB) {
        constexpr int b = decltype(BB)::value;
        static_for<0, NG / 2>([&](auto EE) {
          constexpr int e = 2 * decltype(EE)::value;
          double x[2];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const i32x4& a = acc[b][e + c];
            x[c] = fma(fma((double)a[0], 256.0, (double)a[1]), whi, fma((double)a[2], 256.0, (double)a[3]) * wlo);
          }
          auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x[0]), (unsigned)__double2loint(x[1]), false, false);
          auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x[0]), (unsigned)__double2hiint(x[1]), false, false);
          T[jc * G::kSP + 2 * (e + (g & 1)) + (g >> 1)] = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
        });
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          int row = 4 * u + frw;
          double t = T[row * G::kSP + min(fcol, 2 * NG - 1)];
          *(double*)((char*)(vout + (size_t)(16 * b + 4 * u) * ld) + (unsigned)voff) = ldexp(t * fscale, fex) + fspec;
        }
        __builtin_amdgcn_wave_barrier();
      });
    }
  }
#endif
}

// Geometry of the product for blocks of 17 to 2 NG columns: a wave owns 64 matrix columns, four waves 256.  H = 2: eight waves, each
// with half of the block's columns (one wave with all 16 pairs needs 420 registers, of which half are accumulation registers that every
// matrix instruction's operands have to be copied from: n = 20 000, 32 columns 420 us a product, 332 with two).
template <int NG, int H>
struct WideMM {
  static constexpr int kNJ = 4, kNW = NG / H;                // tiles and pairs per wave
  static constexpr int kThreads = 256 * H;
  static constexpr int kSlotK = 4 * kNJ * 1024;              // a 16-row step of the matrix
  static constexpr int kCopiesK = kNJ / H;
  static constexpr int kRounds = (NG + 4 * H - 1) / (4 * H);
  static constexpr int kSlot = kSlotK + kRounds * 4 * H * 1024;   // and the step's digit record
  static constexpr int kRing = 5;
  static constexpr int kCopies = kCopiesK + kRounds;         // per wave and step
  static constexpr int kFirst = kNW / 4 * kNJ;               // matrix instructions of a step ahead of its barrier
  static_assert(kRing * kSlot <= 160 * 1024 && NG % H == 0 && (H == 1 || kNW == 8), "");
  static_assert(kRounds * 4 * H * 1024 == bbmm_plan::dig_slot_bytes(0, NG), "the last copy of a record may run past it by this much");
};

// out[J] += T^T D[I] for every tile T of the whole matrix, blocks of 17 to 32 columns: 2 NG accumulators a tile for both uses of a tile
// do not fit the registers.  On the fp64 matrix pipe (k_mm_mat, 32 columns) the product is bound by that pipe: 0.45 ms at
// n = 20 000, where reading the matrix takes 0.25.  On words the product takes 0.28 ms with 17 to 24 columns, bound by the reading, and 0.33
// with 32, where a step's reads from LDS (96 KB and 32 KB written) take as long as its matrix instructions.  (Neither a ring of four
// in place of five nor another pitch of the panels changes these.)
// A workgroup takes one strip of 256 columns and one chunk of at most kDigMaxBlocks 16-row steps; sums stay in registers.  Matrix and
// records are copied straight into LDS, four steps ahead.  Behind the first quarter of a step's matrix instructions stand its one
// barrier and then, dealt out behind single instructions, the copies for five steps on and the operands of the next step.
// Workgroups of one XCD take neighbouring strips of the same chunk, so that they share its records in that XCD's L2.
template <int NG, int H>
__global__ __launch_bounds__(256 * H, 1) void k_mm_words_wide(const int* __restrict__ Kw, const char* __restrict__ rec, double* __restrict__ Vp,
                                                          int np, int nsplit, int steps_per_split, const DevState* __restrict__ st) {
#ifdef __HIP_DEVICE_COMPILE__
  if (st->done) return;
  using G = WideMM<NG, H>;
  constexpr int NJ = G::kNJ, NW = G::kNW, LD = 32;
  __shared__ __align__(1024) char lds[G::kRing * G::kSlot];
  lds_char* L0 = (lds_char*)lds;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jc = lane & 15, g = lane >> 4, cw = wave & 3, h = wave >> 2;   // the wave's matrix columns and part of the block
  const int strips = np / 256, nblk = np / 16;               // np is a multiple of 256
  const int w = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // (whole XCDs, see the launch)
  if (w >= strips * nsplit) return;
  const int split = w / strips, strip = w % strips;
  const int ib0 = split * steps_per_split, nk = min(nblk, ib0 + steps_per_split) - ib0;
  double* const vout = Vp + ((size_t)split * np + strip * 256 + cw * (16 * NJ)) * LD;
  if (nk <= 0) {                                             // (a last chunk may be empty: its slot is zero)
    for (int e = h * 64 + lane; e < 16 * NJ * LD; e += 64 * H) vout[e] = 0.0;
    return;
  }
  const int* kb = Kw + ((words_panel_step(strip / 2, np, 1) + ib0) * kWTiles + (strip & 1) * (4 * NJ)) * 256;
  __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)kb, 0, ((nk - 1) * kWTiles + 4 * NJ) * 1024, 0x00020000);
  __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)(rec + (size_t)ib0 * (NG * 1024)), 0,
                                                                (int)bbmm_plan::dig_buffer_bytes(nk, 0, NG), 0x00020000);
  // copy e of step k (past the end the last step comes again: the count of copies stays)
  auto fetch1 = [&](auto EE, int k, int slot) {
    constexpr int e = decltype(EE)::value, c = e - G::kCopiesK;
    if constexpr (e < G::kCopiesK)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (__attribute__((address_space(3))) void*)(L0 + slot + (wave * G::kCopiesK + e) * 1024), 16,
                                               lane * 16, min(k, nk - 1) * (kWTiles * 1024) + (wave * G::kCopiesK + e) * 1024, 0, 2);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rd, (__attribute__((address_space(3))) void*)(L0 + slot + G::kSlotK + (c * 4 * H + wave) * 1024),
                                               16, wave * 1024 + lane * 16, min(k, nk - 1) * (NG * 1024) + c * (4 * H * 1024), 0, 0);
  };
  const int colp = cw * (NJ * 1024) + (g * 16 + (jc ^ g)) * 16, recp = G::kSlotK + h * (NW * 1024) + lane * 16;
  i32x4 acc[NJ][NW], op[2][NW], wk[2][NJ];
#pragma unroll
  for (int b = 0; b < NJ; ++b)
#pragma unroll
    for (int q = 0; q < NW; ++q) acc[b][q] = (i32x4){0, 0, 0, 0};
  // operand o of a step: the matrix words of the wave's tiles, then the record's digits
  auto read1 = [&](auto OO, auto buf, int slot) {
    constexpr int o = decltype(OO)::value;
    if constexpr (o < NJ) wk[decltype(buf)::value][o] = *(lds_i32x4)(L0 + slot + colp + o * 1024);
    else op[decltype(buf)::value][o - NJ] = *(lds_i32x4)(L0 + slot + recp + (o - NJ) * 1024);
  };
  auto next = [](int slot) { return slot + G::kSlot == G::kRing * G::kSlot ? 0 : slot + G::kSlot; };
  static_for<0, G::kRing>([&](auto KK) {
    static_for<0, G::kCopies>([&](auto EE) { fetch1(EE, decltype(KK)::value, decltype(KK)::value * G::kSlot); });
  });
  wait_vm<(G::kRing - 1) * G::kCopies>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  static_for<0, NJ + NW>([&](auto OO) { read1(OO, std::integral_constant<int, 0>{}, 0); });
  int s_cur = 0, s_next = G::kSlot;
  auto step = [&](int k, auto buf) {
    constexpr int B = decltype(buf)::value, M = NJ * NW, M1 = M - G::kFirst;
    static_for<0, M>([&](auto MM) {
      constexpr int m = decltype(MM)::value, q = m / NJ, b = m % NJ, i = m - G::kFirst;
      if constexpr (m == G::kFirst) {
        // This wave's copies of step k + 1 have landed and its reads of step k are done, and so, behind the barrier, are everybody's.
        __builtin_amdgcn_s_waitcnt(0xc07f);
        wait_vm<(G::kRing - 2) * G::kCopies>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      acc[b][q] = mfma_i8(op[B][q], wk[B][b], acc[b][q]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i >= 0) {
        static_for<i * G::kCopies / M1, (i + 1) * G::kCopies / M1>([&](auto EE) { fetch1(EE, k + G::kRing, s_cur); });
        static_for<i * (NJ + NW) / M1, (i + 1) * (NJ + NW) / M1>([&](auto OO) { read1(OO, std::integral_constant<int, 1 - B>{}, s_next); });
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    s_cur = s_next;
    s_next = next(s_next);
  };
#pragma unroll 1
  for (int k = 0; k + 1 < nk; k += 2) {
    step(k, std::integral_constant<int, 0>{});
    step(k + 1, std::integral_constant<int, 1>{});
  }
  if (nk & 1) step(nk - 1, std::integral_constant<int, 0>{});
  __builtin_amdgcn_s_waitcnt(0);                             // copies and reads nobody waited for
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  double* T = (double*)lds + wave * (16 * (LD / H + 1));
#pragma unroll
  for (int b = 0; b < NJ; ++b)
    dig_store<NW, LD / H>(acc[b], 1.0 / (double)kX, T, jc, g, st, vout + (size_t)(16 * b + jc) * LD + h * (LD / H), h * (LD / H));
#endif
}

}  // namespace

size_t words_bytes(int np, bool whole) { return words_panel_step((np + kWP - 1) / kWP, np, whole) * kWTiles * 1024; }

void launch_build_words(hipStream_t s, int kernel, const float* X, int n, int d, int np, int KK, HypArgs hyp, DevState* st,
                        bool whole, double* Xo, double* sqo, int* Kw) {
  k_prep_words<<<(np + 255) / 256, 256, 0, s>>>(X, n, d, np, KK, hyp, st, Xo, sqo);
  dim3 grid((np + kWP - 1) / kWP, (np / 16 + 3) / 4);
  if (kernel == 0) k_build_words<0><<<grid, 256, 0, s>>>(Xo, sqo, n, np, KK, whole, st, Kw);
  else k_build_words<1><<<grid, 256, 0, s>>>(Xo, sqo, n, np, KK, whole, st, Kw);
}

void launch_words_of(hipStream_t s, const float* K, size_t pw, int tri, double outputscale, int n, int np, bool whole, DevState* st, int* Kw) {
  dim3 grid((np + kWP - 1) / kWP, (np / 16 + 3) / 4);
  k_words_of<<<grid, 256, 0, s>>>(K, pw, tri, 1.0 / outputscale, n, np, whole, st, Kw);
}

int launch_mm_words(hipStream_t s, const int* Kw, const void* rec, int ng, double* Vp, int np, int ld, const MmPiece* pieces,
                    const int* first, int wgs, const int* slot_base, const DevState* st) {
  if (ld != 16) return 1;
  switch (ng) {
    case 2: k_mm_words<2><<<wgs, 256, 0, s>>>(Kw, (const char*)rec, Vp, np, ld, pieces, first, slot_base, st); break;
    case 4: k_mm_words<4><<<wgs, 256, 0, s>>>(Kw, (const char*)rec, Vp, np, ld, pieces, first, slot_base, st); break;
    case 6: k_mm_words<6><<<wgs, 256, 0, s>>>(Kw, (const char*)rec, Vp, np, ld, pieces, first, slot_base, st); break;
    default: return 1;
  }
  return 0;
}

int launch_mm_words_wide(hipStream_t s, const int* Kw, const void* rec, int ng, double* Vp, int np, int ld, int nsplit, const DevState* st) {
  int steps = np / 16, per = (steps + nsplit - 1) / nsplit;
  if (ld != 32 || per > kDigMaxBlocks) return 1;
  int grid = (np / 256 * nsplit + 7) / 8 * 8;
  switch (ng) {
    case 9: k_mm_words_wide<9, 1><<<grid, 256, 0, s>>>(Kw, (const char*)rec, Vp, np, nsplit, per, st); break;
    case 12: k_mm_words_wide<12, 1><<<grid, 256, 0, s>>>(Kw, (const char*)rec, Vp, np, nsplit, per, st); break;
    case 16: k_mm_words_wide<16, 2><<<grid, 512, 0, s>>>(Kw, (const char*)rec, Vp, np, nsplit, per, st); break;
    default: return 1;
  }
  return 0;
}
