// FP32 group contractions of the compressed operator (Eqs. 13-14 applied to
// hybrid data) on the FP16 MFMA, every FP32 operand carried as a pair of FP16
// values:
//
//   compress  Z_p[k][y]          = sum_{n,j} A_g[k][n][j] W[n][y][p P + j]
//   expand    W[n][y][p P + j]   = sum_k conj(A_g[k][n][j]) Z_p[k][y]
//
// x s = hi + 2^-11 lo, hi = rn16(x s), lo = rn16(2^11 (x s - hi)), s a power of
// two, is x to half a unit in the last place of FP32 (2^-24); the products hi hi
// and, in an accumulator of their own (their sum takes the 2^-11), hi lo and lo hi
// are summed in FP32 by v_mfma_f32_16x16x32_f16, and lo lo (below 2^-24 of the
// product) is dropped (the two-piece split of Ootomo and Yokota, 2022).  Against
// 64 bits this is closer than the FP32 MFMA: the operands' error is about 2^-24 each,
// and an accumulator is rounded once per 32 products instead of once per two.
// Relative L2 of a contraction of random data against FP64: 1.1-1.6e-7, where
// the FP32 MFMA in its three-multiplication form gives 1.9-3.3e-7 (whole operator
// with K = 520 to 601, forward on pairs 1.8e-7, adjoint on the FP32 MFMA 5.8e-7).  The
// rate is what is bought: three products at 16 times the FP32 MFMA's rate.  On the
// 224 x 224, 32-coil, os 6 slice the two contractions take 24 and 25 us, on the FP32
// MFMA 40 and 43 us.
//
// Scales.  FP16 spans 2^-24 .. 2^16, so every operand is brought under 2^15.  A
// coil's gain is no property of the data (a bank undoes it: noise whitening), so
// coils of very unequal gains are first brought to one size by a power of two c[n]:
// the readout stages take a copy of the maps with it (coils_pair), so that W here is
// c[n] W[n] (compressing) and W[n] / c[n] (expanding), and the bank's columns take
// 1 / c[n].  Then
// - the bank by a power of two per row k of a group (its largest component),
//   applied when the bank is installed; undone in the result of the compressing
//   form, and by Z, in which rows of unequal size meet, in the expanding one;
// - W by a power of two per image row (b, y), from the bound
//   |c[n] W[n][y][t]| <= max_t|psf[y]| / sqrt(Nt) sum_x max_n|c[n] coil[n][y][x]| |img[y][x]|
//   that the readout stage evaluates on the row it transforms anyway;
// - Z^T by a power of two per work-group tile, from the tile's own maximum after
//   that.
// A pair has 24 bits down to 2^-27 of its bound, 22 to 2^-29, and an error of 2^-51 of
// the bound below that, some 2^-20 of what the readout FFT's rounding leaves in a row's
// strongest coil.  Measured, a forward operator's channel that sees one coil only, by
// that coil's size beside the others of its rows: 1.8e-7 down to 2^-20, 2.5e-7 at 2^-24,
// 3.2e-6 at 2^-28; by its entries' size in the bank row: 1.7e-7 at 2^-24, 2.8e-7 at 2^-28,
// 3.2e-6 at 2^-32.
//
// Layouts.  An operand of the MFMA is a "fragment" of 1 KiB: 16 rows x 32
// contraction elements (16 interleaved complex ones), lane (i, h) (i = lane
// % 16, h = lane / 16) holding elements 8h .. 8h + 7 of row i.  The bank is
// stored as fragments (hi, then lo), so a wave reads one with a single
// coalesced 16-byte load per lane and never stages the bank in LDS.  Only the
// row of each expanded pair that gives the real part is stored; the row of
// the imaginary part is (u, v) -> (-v, u) per complex element, exact on the
// pieces, made in registers.
//
// With P odd the (coil, sample) index is padded to an even count per coil
// (PP = P + 1, a zero bank entry), so that a pair of samples, 16 bytes, never
// straddles two coils; 16-byte accesses are then 8-byte aligned.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "devutil.h"
#include "plan.h"

namespace gpjc {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

// Where 16-byte piece (row i, part h) of a fragment of k-block kb lies in LDS,
// in words from the fragment's start.  The XOR spreads the parts, which the
// threads staging a row write at the same time, over the banks: without it
// they lie 256 bytes (64 banks) apart, an eight-way conflict that took two
// thirds of the staging time.
__device__ inline int frag_slot(int i, int h, int kb) { return (h * 16 + (i ^ (4 * h) ^ (2 * (kb & 1)))) * 4; }

constexpr uint32_t kOOBPair = 0x80000000u;
constexpr int kFrag = 256;  // 32-bit words of a fragment

__device__ inline floatx4 mfma16(const floatx4& a, const floatx4& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0,
                                                0);
}

// hi and lo pieces of four scaled values, two per word: three instructions per
// value (v_fma_mixlo / mixhi_f16 for each piece; x s and 2^11 (x s - hi) are
// exact in FP32).  Staging is bound by these.
constexpr float kLo = 2048.f;  // 2^11: lo's scale beside hi's, which keeps lo a normal number as long as hi is one
__device__ inline void split_pair(const floatx4& v, float s, uint2* hi, uint2* lo) {
  uint32_t h[2], l[2];
  const float s2 = s * kLo;
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    half2v hh, ll;
    hh[0] = (_Float16)fmaf(v[2 * w], s, 0.f);
    hh[1] = (_Float16)fmaf(v[2 * w + 1], s, 0.f);
    h[w] = __builtin_bit_cast(uint32_t, hh);
    asm("" : "+v"(h[w]));  // read both halves from here on (else hh[0] is formed twice)
    hh = __builtin_bit_cast(half2v, h[w]);
    ll[0] = (_Float16)fmaf((float)hh[0], -kLo, v[2 * w] * s2);
    ll[1] = (_Float16)fmaf((float)hh[1], -kLo, v[2 * w + 1] * s2);
    l[w] = __builtin_bit_cast(uint32_t, ll);
  }
  *hi = make_uint2(h[0], h[1]);
  *lo = make_uint2(l[0], l[1]);
}

// The other row of an expanded pair: (u, v) -> (-v, u) per complex element.
__device__ inline floatx4 partner(const floatx4& f) {
  floatx4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    r[e] = __uint_as_float(__builtin_rotateleft32(__float_as_uint(f[e]), 16) ^ 0x8000u);
  return r;
}

// Sums of a wave's tile: products hi hi, and hi lo + lo hi (2^11 times as large).
template <int NT>
struct PairAcc {
  floatx4 re[NT], im[NT], rl[NT], il[NT];
  __device__ inline void clear() {
#pragma unroll
    for (int i = 0; i < NT; ++i) re[i] = im[i] = rl[i] = il[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ inline void join() {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      re[i] += rl[i] * (1.f / kLo);
      im[i] += il[i] * (1.f / kLo);
    }
  }
};

// One block of 16 complex contraction elements: a 16-row tile of the bank
// (fragments ah, al of the real part's rows) times NT column tiles whose
// fragments [tile][hi, lo] lie at bs (LDS, this lane's 16 bytes).  A tile's
// fragments are read while the tile before it is multiplied.
template <int NT>
__device__ inline void pair_block(const floatx4& ah, const floatx4& al, const uint32_t* bs, PairAcc<NT>& a) {
  const floatx4 ph = partner(ah), pl = partner(al);
  auto frag = [&](int f) { return *reinterpret_cast<const floatx4*>(bs + f * kFrag); };
  floatx4 bh = frag(0), bl = frag(1);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const floatx4 h = bh, l = bl;
    if (i + 1 < NT) {
      bh = frag(2 * i + 2);
      bl = frag(2 * i + 3);
    }
    a.rl[i] = mfma16(al, h, a.rl[i]);
    a.il[i] = mfma16(pl, h, a.il[i]);
    a.re[i] = mfma16(ah, h, a.re[i]);
    a.im[i] = mfma16(ph, h, a.im[i]);
    a.rl[i] = mfma16(ah, l, a.rl[i]);
    a.il[i] = mfma16(ph, l, a.il[i]);
  }
  // the order above, which the scheduler would undo: two tiles' reads, then
  // six products and two reads in turn
  __builtin_amdgcn_sched_group_barrier(0x100, NT > 1 ? 4 : 2, 0);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
    if (i + 2 < NT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
  }
}

__device__ inline __amdgpu_buffer_rsrc_t pair_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}
__device__ inline floatx4 load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
__device__ inline void store16(__amdgpu_buffer_rsrc_t r, uint32_t off, const floatx4& v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, v), r, (int)off, 0, 0);
}
__device__ inline void store8(__amdgpu_buffer_rsrc_t r, uint32_t off, float2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(uint2v{__float_as_uint(v.x), __float_as_uint(v.y)}, r, (int)off, 0, 0);
}

// old, with the lanes of the 16-lane rows' quarters in BANKS taking src from
// the lane 8 away in the row.
template <int BANKS>
__device__ inline float swap8(float old, float src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, src),
                                                               0x128 /* row_ror:8 */, 0xf, BANKS, false));
}

// a / b for 0 <= a < 2^22, inv = 1.0f / b: (a + 0.5) / b stays 0.5 / b away
// from every integer, more than the rounding of the float product.
__device__ inline int qdiv(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// ---------------------------------------------------------------------------
// Compressing contraction.
//
// Bounds: W is read once (77 MB on the 224 x 224, 32-coil, os 6 slice; HBM /
// Infinity Cache), the MFMA work is 14.8 GFLOP there (6 us at the FP16 peak).
// A work-group takes all rows k of a patch that fit (16 WM complex rows; 80
// at most) and NT tiles of 16 image rows y, so that W is split and staged
// once, and WK wave groups take alternate blocks of a k-tile, so that eight
// waves share one staged tile and the partial sums meet in LDS instead of in
// memory.  k-tiles (16 WK complex values of the (coil, sample) index) are
// fetched into registers two ahead: about 56 KB in flight per CU.  Measured there (5
// tiles, split 2): 24 us, 112 MB moved, 4.7 TB/s, of which the split into pieces and the
// second set of accumulators take about 1.5 us; 64 x 192 x 192, 4.8 GB of W: 1.27 ms.
// ---------------------------------------------------------------------------
struct PairCompress {
  const uint32_t* A;    // bank fragments [G][MT][KB][hi, lo]
  const float2* in;     // [B][nc][N][nt]
  float2* out;          // [ksplit][B][np][K][N]
  const int* pgroup;
  const float* ascale;  // [G][Kp]
  const float* wscale;  // [B][N]
  int MT, KB;           // 16-row tiles of K; 16-element blocks of ns (padded)
  int N, ns, nc, nt, P, PP, np, K, Kp, B, ksplit, tps;  // ns = nc PP (padded); tps: k-tiles per split
  size_t split_stride;
  float invPP;
};

constexpr int pair_wk(int wm) { return wm <= 2 ? 4 : 2; }

template <int WM, int NT, bool ODD>
__global__ __launch_bounds__(64 * WM * pair_wk(WM)) void k_compress_pair(PairCompress a) {
  constexpr int WK = pair_wk(WM), NTHR = 64 * WM * WK;
  constexpr int KT = 16 * WK;    // complex elements per k-tile
  constexpr int CPR = 8 * WK;    // 16-byte chunks per row and k-tile
  constexpr int RPP = NTHR / CPR;  // rows loaded per pass
  constexpr int TN = 16 * NT, R = (TN + RPP - 1) / RPP;
  constexpr int kStage = WK * NT * 2 * kFrag, kRed = (WK - 1) * WM * NT * kFrag;
  __shared__ uint32_t lds[kStage > kRed ? kStage : kRed];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lh = lane >> 4;
  const int wm = wave % WM, wk = wave / WM;
  const int tiles_n = (a.N + TN - 1) / TN, tiles_m = (a.MT + WM - 1) / WM;
  const int logical = xcd_logical(blockIdx.x, tiles_n * tiles_m * a.B * a.np * a.ksplit);
  const int tn = logical % tiles_n;
  const int rest = logical / tiles_n;
  const int tm = rest % tiles_m, z = rest / tiles_m;
  const int ks = z % a.ksplit, bp = z / a.ksplit;
  const int b = bp / a.np, p = bp - b * a.np;
  const int g = a.pgroup[p];
  const int mt = min(tm * WM + wm, a.MT - 1);  // a wave past the last tile repeats it and stores nothing
  const bool mine = tm * WM + wm < a.MT;

  const int ntile = (a.ns + KT - 1) / KT;
  const int t0 = ks * a.tps, t1 = min(ntile, t0 + a.tps);

  // this thread's chunks: elements kk, kk + 1 of rows row0 + RPP r
  const int c = tid % CPR, row0 = tid / CPR;
  const uint32_t rowb = (uint32_t)a.nt * 8u;
  const uint32_t cstride = (uint32_t)a.N * rowb;  // bytes of one coil (host: below 2^31)
  uint32_t roff[R];
  float sc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = row0 + RPP * r, y = tn * TN + row;
    const bool ok = row < TN && y < a.N;
    roff[r] = ok ? (uint32_t)y * rowb : kOOBPair;
    sc[r] = ok ? a.wscale[b * a.N + y] : 1.f;
  }
  const int kend = min(a.ns, t1 * KT);
  int kk = t0 * KT + 2 * c, n = kk / a.PP, j = kk - n * a.PP;
  const float2* in_b = a.in + (size_t)b * a.nc * a.N * a.nt + (size_t)p * a.P;
  uint32_t tail = 0;  // ODD: bit d set if the tile fetched d fetches ago holds padding in this thread's chunks
  // The buffer of a k-tile starts at the coil of the tile's first element, so
  // 32-bit offsets reach every coil the tile touches whatever the size of W.
  auto fetch = [&](int t, floatx4(&x)[R]) {
    const int nf = min((t * KT) / a.PP, a.nc - 1);
    // (ODD: a last pair reaches one sample past the end of W, which is allocated two longer)
    const size_t left = (size_t)(a.nc - nf) * cstride - (size_t)p * a.P * 8 + (ODD ? 8 : 0);
    const __amdgpu_buffer_rsrc_t rw =
        pair_rsrc(in_b + (size_t)nf * a.N * a.nt, (uint32_t)min(left, (size_t)0x7ffffff0));
    const uint32_t off = (uint32_t)(n - nf) * cstride + (uint32_t)j * 8u;
    // out-of-range chunks get offsets of 2^31 and more by an OR, not a select
    // (which the compiler turns into a branch around the load)
    const uint32_t m0 = kk < kend ? 0u : kOOBPair;
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = load16(rw, (off + roff[r]) | m0);
    if (ODD) tail = (tail << 1) | (uint32_t)(j + 1 == a.P);  // the pair's second element is padding
    kk += KT;
    j += KT;
    const int q = qdiv(j, a.invPP);
    j -= q * a.PP;
    n += q;
  };
  const uint32_t* Af = a.A + (((size_t)g * a.MT + mt) * a.KB + wk) * 2 * kFrag + lane * 4;
  auto fetch_bank = [&](int t, floatx4(&f)[2]) {
    const uint32_t* q = Af + (size_t)min(t, ntile - 1) * WK * 2 * kFrag;
    f[0] = *reinterpret_cast<const floatx4*>(q);
    f[1] = *reinterpret_cast<const floatx4*>(q + kFrag);
  };

  // (Kp = 16 MT: rows past K have a scale, and are not stored)
  const floatx4 sa = *reinterpret_cast<const floatx4*>(a.ascale + (size_t)g * a.Kp + 16 * mt + 4 * lh);
  PairAcc<NT> acc;
  acc.clear();
  floatx4(&re)[NT] = acc.re, (&im)[NT] = acc.im;
  floatx4 xw[2][R], xa[2][2];  // two k-tiles ahead
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    fetch(t0 + f, xw[f]);
    fetch_bank(t0 + f, xa[f]);
    __builtin_amdgcn_sched_barrier(0);  // in this order: the loop's first wait counts on it
  }
  const int kbl = c / 8, cc = c % 8;
  uint32_t* const stage = lds + kbl * NT * 2 * kFrag + (cc & 1) * 2;
  const uint32_t* const frags = lds + wk * NT * 2 * kFrag + frag_slot(li, lh, wk);
  auto body = [&](int t, floatx4(&x)[R], floatx4(&f)[2]) {
    __syncthreads();  // the previous k-tile has been read
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + RPP * r;
      if (R * RPP == TN || row < TN) {
        uint2 hi, lo;
        floatx4 v = x[r];
        if (ODD && (tail & 2u)) v[2] = v[3] = 0.f;  // what was read there belongs to the next patch
        split_pair(v, sc[r], &hi, &lo);
        uint32_t* d = stage + (row >> 4) * 2 * kFrag + frag_slot(row & 15, cc >> 1, kbl);
        *reinterpret_cast<uint2*>(d) = hi;
        *reinterpret_cast<uint2*>(d + kFrag) = lo;
      }
    }
    __syncthreads();
    // Issued whether or not there is such a tile (past the end the offsets are
    // out of the buffer's range, so nothing is read): every wait below counts
    // the loads of all paths to it, so a fetch behind a branch, or a way out
    // of the middle of the loop, would make it drain them all.
    fetch(t + 2, x);
    pair_block<NT>(f[0], f[1], frags, acc);
    fetch_bank(t + 2, f);
  };
  int t = t0;
  for (; t + 1 < t1; t += 2) {
    body(t, xw[0], xa[0]);
    body(t + 1, xw[1], xa[1]);
  }
  if (t < t1) body(t, xw[0], xa[0]);
  acc.join();
  // the wave groups' sums, in group order
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    __syncthreads();
    floatx4* red = reinterpret_cast<floatx4*>(lds);
    if (wk > 0) {
#pragma unroll
      for (int i = 0; i < NT; ++i) red[(((wk - 1) * WM + wm) * NT + i) * 64 + lane] = part ? im[i] : re[i];
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int w = 0; w < WK - 1; ++w)
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          const floatx4 v = red[((w * WM + wm) * NT + i) * 64 + lane];
          if (part) im[i] += v;
          else re[i] += v;
        }
    }
  }
  if (wk > 0 || !mine) return;
  float2* out = a.out + ks * a.split_stride + (size_t)bp * a.K * a.N;
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int y = tn * TN + 16 * i + li;
    if (y >= a.N) continue;
    const float uw = pow2_inv(a.wscale[b * a.N + y]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = 16 * mt + 4 * lh + r;
      const float ua = pow2_inv(sa[r]);
      if (k < a.K) out[(size_t)k * a.N + y] = make_float2(re[i][r] * ua * uw, im[i][r] * ua * uw);
    }
  }
}

// ---------------------------------------------------------------------------
// Expanding contraction.
//
// Bounds: W is written once.  A work-group holds the pieces of Z^T for NT
// tiles of 16 image rows and every k in LDS (2 NT KBk KiB), loaded, scaled by
// its own maximum and split once, and its waves walk over tiles of 16 columns
// (n, j), reading the bank's fragments from L2 one step ahead.  Columns lie on
// the rows of the MFMA, permuted so that a lane's registers 0, 1 and 2, 3 are
// neighbouring samples, and neighbouring half-rows of lanes swap halves, so that a
// store instruction writes whole 128-byte segments of W straight from the
// accumulators.  Measured on the 224 x 224, 32-coil, os 6 slice (7 tiles): 25 us, 114 MB,
// 4.5 TB/s; 4.8 GB of W: 1.20 ms.
// ---------------------------------------------------------------------------
struct PairExpand {
  const uint32_t* A;    // bank fragments [G][CT][KBk][hi, lo]
  const float* Zt;      // [B][np][M][2 Kp]
  float2* W;            // [B][nc][M][nt]
  const int* pgroup;
  const float* arel;    // [np][Kp]
  const float* amin;    // [np]
  int CT, KBk;          // 16-column tiles of ns; 16-element blocks of Kp
  int M, Kp, ns, nc, nt, P, PP, np, B, msplit, tps;  // ns = nc PP (padded); tps: column tiles per work-group
  float invPP;
};

template <int NT, int GK, bool MULTI, bool ODD>
__global__ __launch_bounds__(256, 2) void k_expand_pair(PairExpand a) {
  constexpr int TN = 16 * NT;
  // 16-byte chunks of Z^T per thread: 32 / KBk rows at a time, at most 16 times as
  // NT KBk <= 32 (64 KiB)
  constexpr int R = MULTI ? 16 : (TN + 32 / GK - 1) / (32 / GK);
  extern __shared__ uint32_t zs[];  // [KBk][NT][hi, lo] fragments
  float* smax = reinterpret_cast<float*>(zs);  // the waves' maxima, before the fragments
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lh = lane >> 4;
  const int tiles_n = (a.M + TN - 1) / TN;
  const int logical = xcd_logical(blockIdx.x, tiles_n * a.msplit * a.B * a.np);
  const int ms = logical % a.msplit;
  const int rest = logical / a.msplit;
  const int tn = rest % tiles_n, bp = rest / tiles_n;
  const int b = bp / a.np, p = bp - b * a.np;
  const int g = a.pgroup[p];
  const int y0 = tn * TN;
  const int cpr = MULTI ? a.Kp / 2 : 8 * GK;  // chunks per row
  const int nrow = min(TN, a.M - y0);
  const floatx4* src = reinterpret_cast<const floatx4*>(a.Zt + ((size_t)bp * a.M + y0) * 2 * a.Kp);
  const uint32_t* Af = a.A + (size_t)g * a.CT * a.KBk * 2 * kFrag + lane * 4;
  const int c_end = min(a.CT, (ms + 1) * a.tps);
  int ct = ms * a.tps + wave;
  // A step takes GK blocks of k of one column tile (all of them unless MULTI).
  // A block's bank fragments make room for the next step's as soon as they
  // are multiplied, so those are issued before the tile's stores, and waiting
  // for them (loads and stores retire in issue order) never waits for stores.
  const int ng = MULTI ? (a.KBk + GK - 1) / GK : 1;
  floatx4 f[GK][2];
  auto fetch_bank = [&](int tile, int grp, int k) {
    const uint32_t* q =
        Af + ((size_t)min(tile, a.CT - 1) * a.KBk + (MULTI ? min(grp * GK + k, a.KBk - 1) : k)) * 2 * kFrag;
    f[k][0] = *reinterpret_cast<const floatx4*>(q);
    f[k][1] = *reinterpret_cast<const floatx4*>(q + kFrag);
  };
  float sz;
  {
    // chunk c0 of rows row0 + rpp r
    const int rpp = 256 / cpr, row0 = MULTI ? qdiv(tid, 1.f / (float)cpr) : tid / cpr, c0 = tid - row0 * cpr;
    const bool on = row0 < rpp;
    floatx4 x[R];
    float m = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
      x[r] = on && row0 + rpp * r < nrow ? src[tid + rpp * cpr * r] : floatx4{0.f, 0.f, 0.f, 0.f};
    const float2 rel = reinterpret_cast<const float2*>(a.arel + (size_t)p * a.Kp)[c0];
#pragma unroll
    for (int k = 0; k < GK; ++k) fetch_bank(ct, 0, k);
    const floatx4 rk = {rel.x, rel.x, rel.y, rel.y};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      x[r] *= rk;
#pragma unroll
      for (int w = 0; w < 4; ++w) m = fmaxf(m, fabsf(x[r][w]));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if (lane == 0) smax[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]));
    __syncthreads();
    sz = pair_scale(m);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + rpp * r;
      if (on && row < TN) {
        uint2 hi, lo;
        split_pair(x[r], sz, &hi, &lo);
        uint32_t* d = zs + ((c0 >> 3) * NT + (row >> 4)) * 2 * kFrag + frag_slot(row & 15, (c0 & 7) >> 1, c0 >> 3) +
                      (c0 & 1) * 2;
        *reinterpret_cast<uint2*>(d) = hi;
        *reinterpret_cast<uint2*>(d + kFrag) = lo;
      }
    }
  }
  __syncthreads();
  const float ua = pow2_inv(a.amin[p]), uz = pow2_inv(sz);
  const uint32_t rowb = (uint32_t)a.nt * 8u, cstride = (uint32_t)a.M * rowb;  // host: 32-bit offsets reach a tile's coils
  float2* Wb = a.W + (size_t)b * a.nc * a.M * a.nt + (size_t)p * a.P;
  uint32_t roff[2 * NT];
#pragma unroll
  for (int i = 0; i < 2 * NT; ++i) {
    const int y = y0 + 8 * i + (lane & 7);
    roff[i] = y < a.M ? (uint32_t)y * rowb : kOOBPair;
  }
  PairAcc<NT> acc;
  auto store = [&](int tile) {
    acc.join();
    const floatx4(&re)[NT] = acc.re, (&im)[NT] = acc.im;
    // the tile's buffer starts at the coil of its first column; rows and columns out of range are dropped
    const int nf = (16 * tile) / a.PP;
    const size_t left = (size_t)(a.nc - nf) * cstride - (size_t)p * a.P * 8;
    const __amdgpu_buffer_rsrc_t rw =
        pair_rsrc(Wb + (size_t)nf * a.M * a.nt, (uint32_t)min(left, (size_t)0x7ffffff0));
    // Lane (li, lh) holds row li: columns 2 lh (registers 0, 1) and 8 + 2 lh
    // (registers 2, 3).  Lanes li < 8 and li + 8 swap halves, so that an
    // instruction writes whole 16-column (128-byte) segments of eight rows.
    const int col = 16 * tile + ((lane & 8) ? 8 : 0) + 2 * lh;
    const int n = qdiv(col, a.invPP), j = col - n * a.PP;
    const uint32_t off = (uint32_t)(n - nf) * cstride + (uint32_t)j * 8u, m0 = col < a.ns ? 0u : kOOBPair;
    const bool tail = ODD && j + 1 == a.P;
    const uint32_t mt = m0 | (tail ? kOOBPair : 0u);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const floatx4 v0 = floatx4{re[i][0], im[i][0], re[i][1], im[i][1]} * ua * uz;
      const floatx4 v1 = floatx4{re[i][2], im[i][2], re[i][3], im[i][3]} * ua * uz;
      floatx4 lo8, hi8;  // rows li & 7 and 8 + (li & 7)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo8[e] = swap8<0xc>(v0[e], v1[e]);
        hi8[e] = swap8<0x3>(v1[e], v0[e]);
      }
      store16(rw, (off + roff[2 * i]) | mt, lo8);
      store16(rw, (off + roff[2 * i + 1]) | mt, hi8);
      if (tail) {  // the pair's second column is padding
        store8(rw, (off + roff[2 * i]) | m0, make_float2(lo8[0], lo8[1]));
        store8(rw, (off + roff[2 * i + 1]) | m0, make_float2(hi8[0], hi8[1]));
      }
    }
  };
  for (; ct < c_end; ct += 4) {
    acc.clear();
    for (int grp = 0; grp < ng; ++grp) {
      const bool last = grp + 1 == ng;
#pragma unroll
      for (int k = 0; k < GK; ++k) {
        const int kb = MULTI ? grp * GK + k : k;
        if (!MULTI || kb < a.KBk)
          pair_block<NT>(f[k][0], f[k][1], zs + kb * NT * 2 * kFrag + frag_slot(li, lh, kb), acc);
        fetch_bank(last ? ct + 4 : ct, last ? 0 : grp + 1, k);
      }
    }
    store(ct);
  }
}

// ---- bank fragments -----------------------------------------------------------

// Largest component of row blockIdx.x of A_g / c.
__global__ __launch_bounds__(256) void k_pair_max(const double2* __restrict__ A, int nc, int P,
                                                  const float* __restrict__ cscale, float* __restrict__ amax) {
  __shared__ float sh[4];
  const size_t row = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int ns = nc * P;
  const double2* Ak = A + row * ns;
  float m = 0.f;
#pragma unroll 4
  for (int i = threadIdx.x; i < ns; i += 256)
    m = fmaxf(m, fmaxf(fabsf((float)Ak[i].x), fabsf((float)Ak[i].y)) / cscale[i / P]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) amax[row] = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// The scales of patch blockIdx.x's group: ascale[k] brings row k's largest component
// under 2^15; amin is the smallest of them, that of the largest row.  A row of
// zeros, or one past K, takes amin, so that its data keep their size and, being
// multiplied by zeros, cannot set the scale of others: arel is 0 for it.  (arel and
// amin by patch, so that the expanding form reads them with its first loads.)
__global__ __launch_bounds__(256) void k_pair_scales(const float* __restrict__ amax, const int* __restrict__ pgroup,
                                                     int K, int kp, float* __restrict__ ascale,
                                                     float* __restrict__ arel, float* __restrict__ amin) {
  __shared__ float sh[4];
  const int p = blockIdx.x, g = pgroup[p], tid = threadIdx.x;
  const float* m = amax + (size_t)g * K;
  float lo = INFINITY;
  for (int k = tid; k < K; k += 256) lo = m[k] > 0.f ? fminf(lo, pair_scale(m[k])) : lo;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) lo = fminf(lo, __shfl_xor(lo, off, 64));
  if ((tid & 63) == 0) sh[tid >> 6] = lo;
  __syncthreads();
  lo = fminf(fminf(sh[0], sh[1]), fminf(sh[2], sh[3]));
  if (!(lo < INFINITY)) lo = 1.f;
  for (int k = tid; k < kp; k += 256) {
    const bool on = k < K && m[k] > 0.f;
    const float s = on ? pair_scale(m[k]) : lo;
    ascale[(size_t)g * kp + k] = s;  // the same from every patch of the group
    arel[(size_t)p * kp + k] = on ? lo / s : 0.f;
  }
  if (tid == 0) amin[p] = lo;
}

// (s, a power of two, may lie outside the range of a float: the product does not)
__device__ inline void put_pair(uint32_t* frag, int word, float x, float y, double s) {
  uint2 hi, lo;
  split_pair(floatx4{(float)(x * s), (float)(y * s), 0.f, 0.f}, 1.f, &hi, &lo);
  frag[word] = hi.x;
  frag[word + kFrag] = lo.x;
}

// One complex element per thread: words of the compressing fragments [G][MT]
// [KB] (rows k, elements i: conj(A) interleaved), then of the expanding ones
// [G][CT][KBk] (rows c, permuted, elements k: A interleaved), with A / c for A.
// Padding is zero.
__global__ __launch_bounds__(256) void k_pair_bank(const double2* __restrict__ A, const float* __restrict__ cscale,
                                                   const float* __restrict__ ascale,
                                                   uint32_t* __restrict__ Ac, uint32_t* __restrict__ Ae, int G, int K,
                                                   int nc, int P, int PP, int MT, int KB, int CT, int KBk) {
  const size_t cmpw = (size_t)G * MT * KB * kFrag, expw = (size_t)G * CT * KBk * kFrag;
  for (size_t w = (size_t)blockIdx.x * 256 + threadIdx.x; w < cmpw + expw; w += (size_t)gridDim.x * 256) {
    const bool cmp = w < cmpw;
    const size_t v = cmp ? w : w - cmpw;
    const int word = (int)(v % kFrag);
    const size_t f = v / kFrag;
    const int row = (word >> 2) & 15, e = 4 * (word >> 6) + (word & 3);  // row and complex element of the fragment
    int k, i, g;
    if (cmp) {
      i = 16 * (int)(f % KB) + e;
      k = 16 * (int)(f / KB % MT) + row;
      g = (int)(f / KB / MT);
    } else {
      k = 16 * (int)(f % KBk) + e;
      i = 16 * (int)(f / KBk % CT) + 8 * ((row & 3) >> 1) + 2 * (row >> 2) + (row & 1);
      g = (int)(f / KBk / CT);
    }
    const int n = i / PP, j = i - n * PP;  // padded index: j = P is padding where P is odd
    const bool in = k < K && n < nc && j < P;
    const double2 x = in ? A[(((size_t)g * K + k) * nc + n) * P + j] : make_double2(0.0, 0.0);
    const float im = (float)x.y;
    const double s = in ? (double)ascale[(size_t)g * 16 * KBk + k] / cscale[n] : 0.0;  // (Kp = 16 KBk)
    put_pair((cmp ? Ac : Ae) + f * 2 * kFrag, word, (float)x.x, cmp ? -im : im, s);
  }
}

// Set-up, rows y of one work-group: coilmax[y][x], rowp[y], and the row's scales
// set to one (|re| + |im| bounds a modulus; fmaxf drops a NaN, and the row of W that
// it reaches is NaN under any scale); with SIZES, over all rows, each coil's sum of
// the (biased) exponents of its values that are neither zero nor non-finite, and
// their number.  (Integers: the order of the additions does not matter.  A wave
// adds its 64 exponents bit by bit, by ballots, which wait for nothing.)
struct CoilSize {
  unsigned long long sum, count;
};
constexpr int kMaxSizedCoils = 2048;
template <bool SIZES>
__global__ __launch_bounds__(256) void k_pair_setup(const float2* __restrict__ coils, const float2* __restrict__ psf,
                                                    int nc, int nx, int ny, int nt, int B,
                                                    float* __restrict__ coilmax, float* __restrict__ rowp,
                                                    float* __restrict__ wscale, CoilSize* __restrict__ size) {
  __shared__ float sh[4];
  __shared__ unsigned lsum[SIZES ? kMaxSizedCoils : 1], lcnt[SIZES ? kMaxSizedCoils : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  if (SIZES) {
    for (int n = tid; n < nc; n += 256) lsum[n] = lcnt[n] = 0;
    __syncthreads();
  }
  for (int y = blockIdx.x; y < ny; y += gridDim.x) {
    for (int x0 = 0; x0 < nx; x0 += 256) {
      const int x = x0 + tid;
      float m = 0.f;
      for (int n0 = 0; n0 < nc; n0 += 8) {  // eight coils' loads in flight
        float v[8];
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          const float2 c = coils[((size_t)min(n0 + h, nc - 1) * ny + y) * nx + min(x, nx - 1)];
          v[h] = x < nx && n0 + h < nc ? fabsf(c.x) + fabsf(c.y) : 0.f;
        }
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          m = fmaxf(m, v[h]);
          if (SIZES) {
            const int e = (int)(__float_as_uint(v[h]) >> 23);
            const int ok = e < 255 ? e : 0;
            unsigned sum = 0;
#pragma unroll
            for (int b = 0; b < 8; ++b) sum += (unsigned)__popcll(__ballot((ok >> b) & 1)) << b;
            const unsigned cnt = __popcll(__ballot(ok != 0));
            if (lane == 0 && cnt) {
              atomicAdd(&lsum[n0 + h], sum);
              atomicAdd(&lcnt[n0 + h], cnt);
            }
          }
        }
      }
      if (x < nx) coilmax[(size_t)y * nx + x] = m;
    }
    float m = 0.f;
    for (int t = tid; t < nt; t += 256) {
      const float2 v = psf[(size_t)y * nt + t];
      m = fmaxf(m, fabsf(v.x) + fabsf(v.y));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    __syncthreads();
    if (lane == 0) sh[tid >> 6] = m;
    __syncthreads();
    if (tid == 0) rowp[y] = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3])) * rsqrtf((float)nt);
    for (int b = tid; b < B; b += 256) wscale[(size_t)b * ny + y] = 1.f;
  }
  if (SIZES) {
    __syncthreads();
    for (int n = tid; n < nc; n += 256)
      if (lcnt[n]) {
        atomicAdd(&size[n].sum, (unsigned long long)lsum[n]);
        atomicAdd(&size[n].count, (unsigned long long)lcnt[n]);
      }
  }
}

// c[n] from the mean exponents, in steps of 2^16 (a pair has room for less), at most
// 2^64; *unequal is set if any is not one.  A mean: one value of any size does not
// move it.  size NULL: c = 1 throughout.
__global__ __launch_bounds__(256) void k_coil_scale(const CoilSize* __restrict__ size, int nc,
                                                    float* __restrict__ cscale, int* __restrict__ unequal) {
  __shared__ float sh[4];
  const int tid = threadIdx.x;
  auto mean = [&](int n) { return (float)((double)size[n].sum / (double)size[n].count); };
  float most = -INFINITY;
  if (size)
    for (int n = tid; n < nc; n += 256)
      if (size[n].count) most = fmaxf(most, mean(n));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) most = fmaxf(most, __shfl_xor(most, off, 64));
  if ((tid & 63) == 0) sh[tid >> 6] = most;
  __syncthreads();
  most = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
  int any = 0;
  for (int n = tid; n < nc; n += 256) {
    int steps = 0;
    if (size && size[n].count) steps = min((int)((most - mean(n)) / 16.f), 4);
    cscale[n] = __uint_as_float((uint32_t)(127 + 16 * steps) << 23);
    any |= steps;
  }
  any = __syncthreads_or(any);
  if (tid == 0) *unequal = any != 0;
}

// No value of a scaled map above 2^100: one work-group per coil.
__global__ __launch_bounds__(1024) void k_coil_limit(const float2* __restrict__ coils, size_t npix,
                                                     float* __restrict__ cscale) {
  __shared__ int most;
  if (threadIdx.x == 0) most = 0;
  __syncthreads();
  int m = 0;
  for (size_t i = threadIdx.x; i < npix; i += 1024) {
    const float2 c = coils[(size_t)blockIdx.x * npix + i];
    const int e = (int)(__float_as_uint(fabsf(c.x) + fabsf(c.y)) >> 23);
    m = max(m, e < 255 ? e : 0);
  }
  atomicMax(&most, m);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int steps = ((int)(__float_as_uint(cscale[blockIdx.x]) >> 23) - 127) / 16;
    cscale[blockIdx.x] = __uint_as_float((uint32_t)(127 + 16 * min(steps, max(0, (227 - most) / 16))) << 23);
  }
}

__global__ void k_scale_coils(const float2* __restrict__ coils, size_t npix, const float* __restrict__ cscale,
                              float2* __restrict__ out) {
  const float c = cscale[blockIdx.y];
  const size_t base = (size_t)blockIdx.y * npix;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < npix; i += (size_t)gridDim.x * 256)
    out[base + i] = make_float2(coils[base + i].x * c, coils[base + i].y * c);
}

int ceil_div(int n, int d) { return (n + d - 1) / d; }

constexpr int kMaxWM = 5;
int pair_wm(int K) {
  const int mt = ceil_div(K, 16);
  return ceil_div(mt, ceil_div(mt, kMaxWM));
}
// Column tiles at most: as many as leave the accumulators and the loads in flight
// in registers (ten waves have 168 each, the others 256 or more).
constexpr int pair_max_nt(int wm) { return wm == 2 ? 5 : wm == 3 ? 7 : wm == 5 ? 4 : 8; }
int pair_nt(int variant, int wm) { return std::min(8 - variant, pair_max_nt(wm)); }

template <int WM, bool ODD>
void launch_compress_nt(StageScope& sc, hipStream_t s, int nt, const PairCompress& a) {
  constexpr int thr = 64 * WM * pair_wk(WM), N = pair_max_nt(WM);
  const dim3 grid(ceil_div(a.N, 16 * nt) * ceil_div(a.MT, WM) * a.B * a.np * a.ksplit);
  switch (nt) {
    case 1: sc.launch(k_compress_pair<WM, 1, ODD>, grid, dim3(thr), 0, s, a); break;
    case 2: sc.launch(k_compress_pair<WM, 2, ODD>, grid, dim3(thr), 0, s, a); break;
    case 3: sc.launch(k_compress_pair<WM, 3, ODD>, grid, dim3(thr), 0, s, a); break;
    case 4: sc.launch(k_compress_pair<WM, 4, ODD>, grid, dim3(thr), 0, s, a); break;
    case 5: sc.launch(k_compress_pair<WM, std::min(5, N), ODD>, grid, dim3(thr), 0, s, a); break;
    case 6: sc.launch(k_compress_pair<WM, std::min(6, N), ODD>, grid, dim3(thr), 0, s, a); break;
    case 7: sc.launch(k_compress_pair<WM, std::min(7, N), ODD>, grid, dim3(thr), 0, s, a); break;
    default: sc.launch(k_compress_pair<WM, N, ODD>, grid, dim3(thr), 0, s, a); break;
  }
}

template <int WM>
void launch_compress_wm(StageScope& sc, hipStream_t s, int nt, const PairCompress& a) {
  if (a.P & 1) launch_compress_nt<WM, true>(sc, s, nt, a);
  else launch_compress_nt<WM, false>(sc, s, nt, a);
}

constexpr int kMaxGK = 5;  // blocks of k fetched together by the expanding form
template <int GK, bool MULTI, bool ODD>
void launch_expand_nt(StageScope& sc, hipStream_t s, int nt, dim3 grid, uint32_t lds, const PairExpand& a) {
  constexpr int N = MULTI ? 5 : 8;  // with more than kMaxGK blocks of k, at most 5 tiles fit the LDS
  switch (std::min(nt, N)) {
    case 1: sc.launch(k_expand_pair<1, GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    case 2: sc.launch(k_expand_pair<2, GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    case 3: sc.launch(k_expand_pair<3, GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    case 4: sc.launch(k_expand_pair<4, GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    case 5: sc.launch(k_expand_pair<5, GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    case 6: sc.launch(k_expand_pair<std::min(6, N), GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    case 7: sc.launch(k_expand_pair<std::min(7, N), GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
    default: sc.launch(k_expand_pair<N, GK, MULTI, ODD>, grid, dim3(256), lds, s, a); break;
  }
}
template <int GK, bool MULTI>
void launch_expand_gk(StageScope& sc, hipStream_t s, int nt, dim3 grid, uint32_t lds, const PairExpand& a) {
  if (a.P & 1) launch_expand_nt<GK, MULTI, true>(sc, s, nt, grid, lds, a);
  else launch_expand_nt<GK, MULTI, false>(sc, s, nt, grid, lds, a);
}

constexpr int kExpandLds = 65536;  // bytes of Z^T pieces per work-group

}  // namespace

static int pair_pp(const Plan& pl) { return pl.P + (pl.P & 1); }
static int pair_ns(const Plan& pl) { return pl.nc * pair_pp(pl); }
static int pair_kblocks(int ns) { return ceil_div(ns, 64) * 4; }  // blocks of 16, whole k-tiles of either WK
size_t place_pair_scales(Plan& pl) {
  float* p = pl.scales;
  size_t used = 0;
  auto take = [&](float** a, size_t n) {
    *a = p ? p + used : nullptr;
    used += (n + 63) / 64 * 64;
  };
  take(&pl.wscale, (size_t)pl.B * pl.ny);
  take(&pl.cscale, pl.nc);
  take(&pl.coilsize, sizeof(CoilSize) / sizeof(float) * (size_t)pl.nc);
  float* flag = nullptr;
  take(&flag, 1);
  pl.unequal = reinterpret_cast<int*>(flag);
  take(&pl.coilmax, (size_t)pl.ny * pl.nx);
  take(&pl.rowp, pl.ny);
  take(&pl.ascale, (size_t)pl.G * pl.Kp);
  take(&pl.arel, (size_t)pl.np * pl.Kp);
  take(&pl.amin, pl.np);
  take(&pl.amax, (size_t)pl.G * pl.K);
  return used;
}
size_t pair_compress_words(const Plan& pl) {
  return (size_t)pl.G * ceil_div(pl.K, 16) * pair_kblocks(pair_ns(pl)) * 2 * kFrag;
}
size_t pair_expand_words(const Plan& pl) {
  return (size_t)pl.G * ceil_div(pair_ns(pl), 16) * (pl.Kp / 16) * 2 * kFrag;
}

// 32-bit offsets within a k-tile, which touches at most KT / P + 2 coils.
bool pair_compress_ok(const Plan& pl) {
  const int kt = 16 * pair_wk(pair_wm(pl.K));
  return (size_t)(kt / pl.P + 2) * pl.ny * pl.nt * 8 < kOOBPair;
}
bool pair_expand_ok(const Plan& pl) {
  return (pl.Kp / 16) * 2048 <= kExpandLds && pair_ns(pl) < (1 << 22) &&
         (size_t)(16 / pl.P + 2) * pl.ny * pl.nt * 8 < kOOBPair;
}

// Coil maps within 2^16 of each other, which is all but a set-up of very unequal
// gains, keep c = 1 and need no copy.  The others get one by scale_coils, once the
// stream has run and *unequal is known.
int setup_pair(Plan& pl) {
  const bool sizes = pl.nc <= kMaxSizedCoils;
  CoilSize* size = reinterpret_cast<CoilSize*>(pl.coilsize);
  pl.coils_pair = pl.coils;
  const dim3 grid(std::min(pl.ny, 1024));
  if (sizes) {
    GPJC_HIP(hipMemsetAsync(size, 0, sizeof(CoilSize) * pl.nc, pl.stream));
    hipLaunchKernelGGL(k_pair_setup<true>, grid, dim3(256), 0, pl.stream, pl.coils, pl.psf, pl.nc, pl.nx, pl.ny, pl.nt,
                       pl.B, pl.coilmax, pl.rowp, pl.wscale, size);
  } else {
    hipLaunchKernelGGL(k_pair_setup<false>, grid, dim3(256), 0, pl.stream, pl.coils, pl.psf, pl.nc, pl.nx, pl.ny,
                       pl.nt, pl.B, pl.coilmax, pl.rowp, pl.wscale, size);
  }
  hipLaunchKernelGGL(k_coil_scale, dim3(1), dim3(256), 0, pl.stream, sizes ? size : nullptr, pl.nc, pl.cscale,
                     pl.unequal);
  GPJC_HIP(hipGetLastError());
  return GPJC_OK;
}

int scale_coils(Plan& pl) {
  const size_t npix = (size_t)pl.ny * pl.nx;
  float2* p = nullptr;
  GPJC_HIP(hipMalloc(reinterpret_cast<void**>(&p), sizeof(float2) * pl.nc * npix));
  pl.coils_pair = p;
  hipLaunchKernelGGL(k_coil_limit, dim3(pl.nc), dim3(1024), 0, pl.stream, pl.coils, npix, pl.cscale);
  hipLaunchKernelGGL(k_scale_coils, dim3((unsigned)std::min<size_t>((npix + 255) / 256, 1024), pl.nc), dim3(256), 0,
                     pl.stream, pl.coils, npix, pl.cscale, p);
  hipLaunchKernelGGL(k_pair_setup<false>, dim3(std::min(pl.ny, 1024)), dim3(256), 0, pl.stream, pl.coils_pair, pl.psf,
                     pl.nc, pl.nx, pl.ny, pl.nt, pl.B, pl.coilmax, pl.rowp, pl.wscale, nullptr);
  GPJC_HIP(hipGetLastError());
  GPJC_HIP(hipStreamSynchronize(pl.stream));
  return GPJC_OK;
}

int launch_pair_bank(const Plan& pl) {
  hipLaunchKernelGGL(k_pair_max, dim3(pl.K, pl.G), dim3(256), 0, pl.stream, pl.A128, pl.nc, pl.P, pl.cscale, pl.amax);
  hipLaunchKernelGGL(k_pair_scales, dim3(pl.np), dim3(256), 0, pl.stream, pl.amax, pl.pgroup, pl.K, pl.Kp, pl.ascale,
                     pl.arel, pl.amin);
  const size_t words = (pair_compress_words(pl) + pair_expand_words(pl)) / 2;
  hipLaunchKernelGGL(k_pair_bank, dim3((unsigned)std::min<size_t>((words + 255) / 256, 8192)), dim3(256), 0, pl.stream,
                     pl.A128, pl.cscale, pl.ascale, pl.Ac2, pl.Ae2, pl.G, pl.K, pl.nc, pl.P, pair_pp(pl),
                     ceil_div(pl.K, 16), pair_kblocks(pair_ns(pl)), ceil_div(pair_ns(pl), 16), pl.Kp / 16);
  GPJC_HIP(hipGetLastError());
  return GPJC_OK;
}

// Work-groups of one split.
static long pair_groups(const Plan& pl, int nt) {
  return (long)ceil_div(pl.ny, 16 * nt) * ceil_div(ceil_div(pl.K, 16), pair_wm(pl.K)) * pl.B * pl.np;
}

// Column tiles of the expanding form: the largest count that fits the LDS and
// pads the rows by at most an eighth (a larger one reads the bank less often, and
// writes W in longer runs for the readout stage to read), then smaller ones while the
// launch cannot give every CU a work-group with a column tile per wave.  Measured for
// 4 and 8 tiles, a whole operator, us: 32 x 64 rows of 48, K = 12, 191 and 185; 2 x 230 rows
// of 180, K = 24, encode and adjoint, 180 and 183; W of 4.8 GB, the kernel alone, 1322 and
// 1192.
static int pair_expand_tiles(const Plan& pl) {
  const int n = ceil_div(pl.ny, 16), ct = ceil_div(pair_ns(pl), 16);
  int t = std::min(n, std::max(1, std::min(8, kExpandLds / (2048 * (pl.Kp / 16)))));
  while (t > 1 && 8 * ceil_div(n, t) * t > 9 * n) --t;
  while (t > 1 && (long)ceil_div(n, t) * pl.B * pl.np * ceil_div(ct, 4) < 256) --t;
  return t;
}

// Work-groups of the compressing form resident per CU, by registers.
static int pair_resident(int wm, int nt) {
  static const uint8_t kRes[kMaxWM][5] = {
      {4, 3, 2, 2, 1}, {3, 2, 1, 1, 1}, {3, 2, 2, 2, 1}, {2, 2, 1, 1, 1}, {2, 1, 1, 1, 1}};
  return kRes[wm - 1][std::min(nt, 5) - 1];
}

// Column tiles and split of the compressing form by the time they are
// expected to take: a work-group needs about 2 us to fill and drain and 0.15 + 0.18
// NT us (for WK = 2) per k-tile, half as long again for each work-group that
// shares the CU, the launch as many such rounds as its work-groups make, and every
// split writes and reads back a partial of Z at about 5 TB/s.  No split where the
// launch has four work-groups per CU without one: there it adds partials of Z and no
// parallelism.  Measured (kernel alone, us), 224 x 224, 32-coil slice, splits of 1, 2, 3:
// 7 tiles 45, 29, 25; 5 tiles 36, 25, 34; 3 tiles 28, 30, 32; one split: 2 x 230 rows of
// 180, P = 15, K = 24, 1, 2, 3, 4, 6 tiles: 33.5, 31.8, 36.0, 39.1, 43.8; 4 x 112 rows, K = 30:
// 19.7, 16.4, 21.9, 18.9, 27.5; 64 x 192 rows, K = 56: 1869, 1486, 1466, 1564, 1444 (8: 1325).
void default_pair_compress(const Plan& pl, Plan::GemmCfg& g) {
  const int n = ceil_div(pl.ny, 16), wm = pair_wm(pl.K), wk = pair_wk(wm), ntile = ceil_div(pair_ns(pl), 16 * wk);
  const double zus = 16.0 * pl.K * pl.ny * pl.np * pl.B / 5e6;
  double best = 1e30;
  g.ksplit = 1;
  g.cvar = 0;
  for (int t = std::min(n, pair_max_nt(wm)); t >= 1; --t) {
    const long groups = pair_groups(pl, t);
    const int res = pair_resident(wm, t), most = groups >= 1024 ? 1 : std::min(kMaxKsplit, ntile);
    for (int ks = 1; ks <= most; ++ks) {
      const long per_cu = (groups * ks + 255) / 256, rem = per_cu % res;
      const double rounds = per_cu / res * (0.5 + 0.5 * res) + (rem ? 0.5 + 0.5 * rem : 0.0);
      const double us = rounds * (ceil_div(ntile, ks) * (0.15 + 0.18 * t) * wk / 2 + 2.0) + zus * ks + 0.3 * (ks - 1);
      if (us < best) {
        best = us;
        g.cvar = 8 - t;
        g.ksplit = ks;
      }
    }
  }
}
void default_pair_expand(const Plan& pl, Plan::GemmCfg& g) { g.evar = 8 - pair_expand_tiles(pl); }

// The variants below these run as they do: fewer column tiles than their number says.
int pair_first_compress(const Plan& pl) { return 8 - pair_max_nt(pair_wm(pl.K)); }
int pair_first_expand(const Plan& pl) {
  const int kbk = pl.Kp / 16;
  return 8 - std::min(kbk > kMaxGK ? 5 : 8, kExpandLds / (2048 * kbk));
}

// Partials of Z that a split leaves: 1 where the launch has four work-groups per CU
// without one (a tuned choice of a smaller plan's bucket, or a caller's).
int pair_partials(const Plan& pl, const Plan::GemmCfg& cfg) {
  return pair_groups(pl, pair_nt(cfg.cvar, pair_wm(pl.K))) >= 1024 ? 1 : cfg.ksplit;
}

int launch_compress_pair(const Plan& pl, StageScope& sc, const void* in, float2* out) {
  const Plan::GemmCfg& cfg = pl.cfg(Store::F32);
  const int wm = pair_wm(pl.K), nt = pair_nt(cfg.cvar, wm), kt = 16 * pair_wk(wm);
  PairCompress a{};
  a.A = pl.Ac2;
  a.in = static_cast<const float2*>(in);
  a.out = out;
  a.pgroup = pl.pgroup;
  a.ascale = pl.ascale;
  a.wscale = pl.wscale;
  a.MT = ceil_div(pl.K, 16);
  a.KB = pair_kblocks(pair_ns(pl));
  a.N = pl.ny;
  a.ns = pair_ns(pl);
  a.nc = pl.nc;
  a.nt = pl.nt;
  a.P = pl.P;
  a.PP = pair_pp(pl);
  a.np = pl.np;
  a.K = pl.K;
  a.Kp = pl.Kp;
  a.B = pl.B;
  a.ksplit = pair_partials(pl, cfg);
  a.tps = ceil_div(ceil_div(a.ns, kt), a.ksplit);
  a.split_stride = (size_t)pl.B * pl.np * pl.K * pl.ny;
  a.invPP = 1.f / (float)a.PP;
  switch (wm) {
    case 1: launch_compress_wm<1>(sc, pl.stream, nt, a); break;
    case 2: launch_compress_wm<2>(sc, pl.stream, nt, a); break;
    case 3: launch_compress_wm<3>(sc, pl.stream, nt, a); break;
    case 4: launch_compress_wm<4>(sc, pl.stream, nt, a); break;
    default: launch_compress_wm<5>(sc, pl.stream, nt, a); break;
  }
  GPJC_HIP(hipGetLastError());
  return GPJC_OK;
}

int launch_expand_pair(const Plan& pl, StageScope& sc) {
  const int kbk = pl.Kp / 16;
  const int nt = std::max(1, std::min(8 - pl.cfg(Store::F32).evar, kExpandLds / (2048 * kbk)));
  PairExpand a{};
  a.A = pl.Ae2;
  a.Zt = reinterpret_cast<const float*>(pl.Zt);
  a.W = pl.W;
  a.pgroup = pl.pgroup;
  a.arel = pl.arel;
  a.amin = pl.amin;
  a.CT = ceil_div(pair_ns(pl), 16);
  a.KBk = kbk;
  a.M = pl.ny;
  a.Kp = pl.Kp;
  a.ns = pair_ns(pl);
  a.nc = pl.nc;
  a.nt = pl.nt;
  a.P = pl.P;
  a.PP = pair_pp(pl);
  a.np = pl.np;
  a.B = pl.B;
  a.invPP = 1.f / (float)a.PP;
  // as many work-groups as are resident at once (by LDS, and by registers: at most
  // 128 up to 2 tiles, 168 up to 4, or 5 with at most 3 blocks of k to a step), but a
  // column tile per wave; on the 224 x 224, 32-coil slice 7 tiles with 504 work-groups
  // take 21.8 us, with 672, not all resident, 27.0 us
  const int base = ceil_div(pl.ny, 16 * nt) * pl.B * pl.np;
  const int gk = ceil_div(kbk, ceil_div(kbk, kMaxGK));
  const int occ = std::min(nt <= 2 ? 4 : nt <= 4 || (nt == 5 && gk <= 3) ? 3 : 2, 163840 / (kbk * nt * 2048));
  const int ms = std::max(1, std::min(256 * occ / base, ceil_div(a.CT, 4)));
  a.tps = ceil_div(a.CT, ms);
  a.msplit = ceil_div(a.CT, a.tps);
  const dim3 grid(base * a.msplit);
  const uint32_t lds = (uint32_t)(kbk * nt * 2048);
  const bool multi = kbk > kMaxGK;
  switch (gk) {
    case 1: launch_expand_gk<1, false>(sc, pl.stream, nt, grid, lds, a); break;
    case 2: launch_expand_gk<2, false>(sc, pl.stream, nt, grid, lds, a); break;
    case 3:
      if (multi) launch_expand_gk<3, true>(sc, pl.stream, nt, grid, lds, a);
      else launch_expand_gk<3, false>(sc, pl.stream, nt, grid, lds, a);
      break;
    case 4:
      if (multi) launch_expand_gk<4, true>(sc, pl.stream, nt, grid, lds, a);
      else launch_expand_gk<4, false>(sc, pl.stream, nt, grid, lds, a);
      break;
    default:
      if (multi) launch_expand_gk<5, true>(sc, pl.stream, nt, grid, lds, a);
      else launch_expand_gk<5, false>(sc, pl.stream, nt, grid, lds, a);
      break;
  }
  GPJC_HIP(hipGetLastError());
  return GPJC_OK;
}

}  // namespace gpjc
