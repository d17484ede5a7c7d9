// LDS-resident Stockham FFT for batches of power-of-two sequences.
//
// Each stage of radix R with current sub-transform length Ns reads input
// j + r (M/R), applies the twiddle w^(r k), k = j mod Ns, w = exp(s 2 pi i /
// (Ns R)), does a radix-R DFT in registers and writes output
// (j / Ns) Ns R + k + r Ns (the autosorting Stockham ordering), so the result
// is in natural order without a bit-reversal pass.  Stages: one radix-2^(p mod
// 4) stage first (no twiddles) when p = log2 M is not a multiple of 4, then
// radix-16 stages.  Twiddles exp(+2 pi i t / M) come from a two-level table
// held in LDS: lo[t mod 64] * hi[t / 64], lo[q] = exp(2 pi i q / M) and
// hi[q] = exp(2 pi i 64 q / M), both computed in FP64 on the host and rounded
// once (one extra rounding per twiddle).
#pragma once

#include "common.h"

namespace pc {

template <typename R>
__host__ __device__ __forceinline__ cpx<R> cmul(cpx<R> a, cpx<R> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// exp(SIGN 2 pi i K / N) applied to v, with exact handling of the trivial
// angles (multiples of pi/2) so that no multiplication by 0/1 is emitted.
template <typename R, int N, int SIGN>
__host__ __device__ __forceinline__ cpx<R> rot(cpx<R> v, int K) {
  // cos(2 pi q / 16) for q = 0..4 (first quadrant), as literals so that no
  // table is materialised
  auto c16 = [](int q) -> double {
    return q == 0 ? 1.0
                  : q == 1 ? 0.92387953251128675613
                           : q == 2 ? 0.70710678118654752440
                                    : q == 3 ? 0.38268343236508977173 : 0.0;
  };
  const int k16 = (K * 16 / N) & 15;  // angle in units of 2 pi / 16
  if (k16 == 0) return v;
  if (k16 == 4) return SIGN > 0 ? cpx<R>{-v.y, v.x} : cpx<R>{v.y, -v.x};
  if (k16 == 8) return {-v.x, -v.y};
  if (k16 == 12) return SIGN > 0 ? cpx<R>{v.y, -v.x} : cpx<R>{-v.y, v.x};
  const int q = k16 & 3, quad = k16 >> 2;
  R c = (R)c16(q), s = (R)c16(4 - q);
  // rotate (c, s) by quad quarter turns
  for (int t = 0; t < quad; ++t) {
    R nc = -s, ns = c;
    c = nc;
    s = ns;
  }
  if (SIGN < 0) s = -s;
  return {v.x * c - v.y * s, v.x * s + v.y * c};
}

// In-register DFT of length N (N = 2, 4, 8, 16) with sign SIGN, radix-2 DIT.
template <typename R, int N, int SIGN>
__host__ __device__ __forceinline__ void dft(cpx<R>* x) {
  if constexpr (N == 1) {
    return;
  } else if constexpr (N == 2) {
    cpx<R> a = x[0], b = x[1];
    x[0] = {a.x + b.x, a.y + b.y};
    x[1] = {a.x - b.x, a.y - b.y};
  } else {
    cpx<R> e[N / 2], o[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      e[i] = x[2 * i];
      o[i] = x[2 * i + 1];
    }
    dft<R, N / 2, SIGN>(e);
    dft<R, N / 2, SIGN>(o);
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
      cpx<R> t = rot<R, N, SIGN>(o[k], k);
      x[k] = {e[k].x + t.x, e[k].y + t.y};
      x[k + N / 2] = {e[k].x - t.x, e[k].y - t.y};
    }
  }
}

constexpr int ilog2(int m) { return m <= 1 ? 0 : 1 + ilog2(m / 2); }
constexpr int first_radix(int m) { return (ilog2(m) % 4) ? (1 << (ilog2(m) % 4)) : 16; }

// Entries of the two-level twiddle table for a transform of length M.
__host__ __device__ constexpr int tw_hi_count(int m) { return m / 64 > 1 ? m / 64 : 1; }
__host__ __device__ constexpr int tw_count(int m) { return 64 + tw_hi_count(m); }

// Copies the two-level table from global memory into LDS (all threads; ends
// with a barrier).
template <typename R, int M, int NT>
__device__ __forceinline__ void load_twiddles(cpx<R>* lds, const cpx<R>* __restrict__ tw) {
  for (int i = threadIdx.x; i < tw_count(M); i += NT) lds[i] = tw[i];
  __syncthreads();
}

// LDS position of element i of the FFT buffers: one padding slot after every
// 16 elements, so that the power-of-two strides of the Stockham stages do not
// map all lanes of a wave onto the same banks.
__host__ __device__ constexpr int pidx(int i) { return i + (i >> 4); }
__host__ __device__ constexpr int padded(int n) { return n + (n >> 4); }

template <typename R, int M>
__device__ __forceinline__ cpx<R> twiddle(const cpx<R>* tws, int t) {
  return cmul(tws[t & 63], tws[64 + (t >> 6)]);
}

// Radix-2 butterfly with twiddle t in fused multiply-adds:
// (a, b) <- (a + t b, a - t b), the difference formed as 2a - (a + t b)
// (six instructions instead of a product, a sum and a difference).
template <typename R>
__host__ __device__ __forceinline__ R fmar(R a, R b, R c) {
  if constexpr (sizeof(R) == 4)
    return __builtin_fmaf(a, b, c);
  else
    return __builtin_fma(a, b, c);
}

template <typename R>
__host__ __device__ __forceinline__ void bfly_tw(cpx<R>& a, cpx<R>& b, cpx<R> t) {
  const cpx<R> p = {fmar(t.x, b.x, fmar(-t.y, b.y, a.x)), fmar(t.x, b.y, fmar(t.y, b.x, a.y))};
  b = {fmar(R(2), a.x, -p.x), fmar(R(2), a.y, -p.y)};
  a = p;
}

// u^2 for u of modulus one up to rounding, as (1 - 2 y^2, 2 x y).  The product
// u u would double the modulus' error with each squaring; here the cosine comes
// from the sine, which for the angles of a stage's own twiddles (up to 1/16
// turn) is the more accurate of the two.
template <typename R>
__host__ __device__ __forceinline__ cpx<R> unit_square(cpx<R> u) {
  const R t = u.y + u.y;
  return {fmar(-t, u.y, R(1)), t * u.x};
}

// Twiddled DFT of length N (a power of two) in registers:
// x[f] <- sum_r x[r] (u exp(SIGN 2 pi i f / N))^r, the input twiddles u^r of a
// Stockham stage folded into the transform.  Splitting r into even and odd
// gives two twiddled DFTs of length N/2 with twiddle u^2, joined by
// butterflies with t_f = u exp(SIGN 2 pi i f / N) (t_{f + N/4} = t_f i^SIGN),
// so the stage costs log2(N) squarings and a few constant rotations of u
// instead of N - 2 products forming the powers and N - 1 applying them.
template <typename R, int N, int SIGN>
__host__ __device__ __forceinline__ void dft_tw(cpx<R>* x, cpx<R> u) {
  if constexpr (N > 1) {
    cpx<R> e[N / 2], o[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      e[i] = x[2 * i];
      o[i] = x[2 * i + 1];
    }
    if constexpr (N > 2) {
      const cpx<R> u2 = unit_square(u);
      dft_tw<R, N / 2, SIGN>(e, u2);
      dft_tw<R, N / 2, SIGN>(o, u2);
    }
    cpx<R> t[N / 2];
#pragma unroll
    for (int f = 0; f < N / 2; ++f) {
      if (N == 2 || f < N / 4) {
        t[f] = rot<R, N, SIGN>(u, f);
      } else {
        const cpx<R> v = t[f - N / 4];
        t[f] = SIGN > 0 ? cpx<R>{-v.y, v.x} : cpx<R>{v.y, -v.x};
      }
    }
#pragma unroll
    for (int f = 0; f < N / 2; ++f) {
      bfly_tw(e[f], o[f], t[f]);
      x[f] = e[f];
      x[f + N / 2] = o[f];
    }
  }
}

template <typename R, int RAD, int M, int NB, int NT, int SIGN, int NS>
__device__ __forceinline__ void fft_stage(cpx<R>* buf, const cpx<R>* tw) {
  constexpr int NBF = M / RAD;
  constexpr int TOT = NB * NBF;
  constexpr int PER = (TOT + NT - 1) / NT;
  // padded positions of the stage's strided reads and writes: when the
  // stride is a multiple of 16 the padding adds a constant per step
  constexpr bool RD_LIN = NBF % 16 == 0;
  constexpr bool WR_LIN = NS % 16 == 0;
  cpx<R> y[PER][RAD];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int bi = (int)threadIdx.x + q * NT;
    if (TOT % NT == 0 || bi < TOT) {
      const int b = bi / NBF, j = bi - b * NBF;
      const int k = j & (NS - 1);
      cpx<R> x[RAD];
      const int i0 = b * M + j;
#pragma unroll
      for (int r = 0; r < RAD; ++r)
        x[r] = RD_LIN ? buf[pidx(i0) + r * padded(NBF)] : buf[pidx(i0 + r * NBF)];
      if constexpr (NS > 1) {
        cpx<R> w1 = twiddle<R, M>(tw, k * (M / (NS * RAD)));
        if (SIGN < 0) w1.y = -w1.y;
        dft_tw<R, RAD, SIGN>(x, w1);
      } else {
        dft<R, RAD, SIGN>(x);
      }
#pragma unroll
      for (int r = 0; r < RAD; ++r) y[q][r] = x[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int bi = (int)threadIdx.x + q * NT;
    if (TOT % NT == 0 || bi < TOT) {
      const int b = bi / NBF, j = bi - b * NBF;
      const int k = j & (NS - 1);
      const int base = b * M + (j / NS) * NS * RAD + k;
#pragma unroll
      for (int r = 0; r < RAD; ++r) {
        if (WR_LIN)
          buf[pidx(base) + r * padded(NS)] = y[q][r];
        else
          buf[pidx(base + r * NS)] = y[q][r];
      }
    }
  }
  __syncthreads();
}

template <typename R, int M, int NB, int NT, int SIGN, int NS>
__device__ __forceinline__ void fft_stages(cpx<R>* buf, const cpx<R>* tw) {
  if constexpr (NS < M) {
    constexpr int RAD = (NS == 1) ? first_radix(M) : 16;
    fft_stage<R, RAD, M, NB, NT, SIGN, NS>(buf, tw);
    fft_stages<R, M, NB, NT, SIGN, NS * RAD>(buf, tw);
  }
}

// The last stage (NS * RAD = M), with each output handed to store(b, f, v)
// (f = frequency index of sequence b) from registers instead of written back
// to LDS, for the outputs keep(f) selects (for RAD = 16 and a keep that tests
// ranges of M / 16, decided per r at compile time).  Butterflies j (outputs
// j + r NS) for which need(j) is false are skipped whole.  No barrier at the
// end.
struct AllNeeded {
  __device__ bool operator()(int) const { return true; }
};

template <typename R, int RAD, int M, int NB, int NT, int SIGN, int NS, typename Keep,
          typename Store, typename Need = AllNeeded>
__device__ __forceinline__ void fft_last_stage(const cpx<R>* buf, const cpx<R>* tw, Keep keep,
                                               Store store, Need need = Need{}) {
  static_assert(NS * RAD == M, "last stage");
  constexpr int NBF = M / RAD;  // == NS: j is its own twiddle index
  constexpr int TOT = NB * NBF;
  constexpr int PER = (TOT + NT - 1) / NT;
  constexpr bool RD_LIN = NBF % 16 == 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int bi = (int)threadIdx.x + q * NT;
    if (TOT % NT == 0 || bi < TOT) {
      const int b = bi / NBF, j = bi - b * NBF;
      if (!need(j)) continue;
      cpx<R> x[RAD];
      const int i0 = b * M + j;
#pragma unroll
      for (int r = 0; r < RAD; ++r)
        x[r] = RD_LIN ? buf[pidx(i0) + r * padded(NBF)] : buf[pidx(i0 + r * NBF)];
      if constexpr (NS > 1) {
        cpx<R> w1 = twiddle<R, M>(tw, j);
        if (SIGN < 0) w1.y = -w1.y;
        dft_tw<R, RAD, SIGN>(x, w1);
      } else {
        dft<R, RAD, SIGN>(x);
      }
#pragma unroll
      for (int r = 0; r < RAD; ++r) {
        const int f = r * NS + j;
        if (keep(r, f)) store(b, f, x[r]);
      }
    }
  }
}

template <typename R, int M, int NB, int NT, int SIGN, int NS, typename Keep, typename Store,
          typename Need>
__device__ __forceinline__ void fft_stages_store(cpx<R>* buf, const cpx<R>* tw, Keep keep,
                                                 Store store, Need need) {
  constexpr int RAD = (NS == 1) ? first_radix(M) : 16;
  if constexpr (NS * RAD < M) {
    fft_stage<R, RAD, M, NB, NT, SIGN, NS>(buf, tw);
    fft_stages_store<R, M, NB, NT, SIGN, NS * RAD>(buf, tw, keep, store, need);
  } else {
    fft_last_stage<R, RAD, M, NB, NT, SIGN, NS>(buf, tw, keep, store, need);
  }
}

// FFT of NB sequences in LDS from stage NS on, the last stage's outputs
// stored through store(b, f, v) for keep(r, f), its butterflies j run only
// where need(j) (see fft_last_stage); the LDS contents are left undefined.
template <typename R, int M, int NB, int NT, int SIGN, int NS = 1, typename Keep, typename Store,
          typename Need = AllNeeded>
__device__ __forceinline__ void lds_fft_store(cpx<R>* buf, const cpx<R>* tw, Keep keep,
                                              Store store, Need need = Need{}) {
  fft_stages_store<R, M, NB, NT, SIGN, NS>(buf, tw, keep, store, need);
}

// ---------------------------------------------------------------------------
// Register-held transforms of length M = 4096 S (S = 1, 2, 4) whose input
// lies in a window of 4096 consecutive slots centred on M / 2 (any 4096 slots
// are the whole input for S = 1), FP32, one sequence per 256 threads.
//
// The outputs f = S k + s of one residue s are a 4096-point transform of the
// input with its own twiddles, X[S k + s] = sum_m x_m w^(m (S k + s)),
// w = exp(SIGN 2 pi i / M): thread t holds the inputs of slots t + 256 r (mod
// 4096), r < 16, in registers for all residues, and three radix-16 stages with
// twiddles u_1 = w^(256 s), u_2 = w^(16 (S k_1 + s)), u_3 = w^(S (k_1 + 16
// k_2) + s) (folded into the DFTs, see dft_tw) give k = k_1 + 16 k_2 + 256 k_3;
// the zero input slots cost nothing, no full-length buffer is needed, and two
// LDS exchanges per residue replace the four of a padded length-M transform.
// Slots at or above M / 2 (r < 8) carry w^(4096 S/2 s), those below
// w^(4096 (S/2 - 1) s): quarter or half turns known at compile time.
// 36 to 39 KB of LDS with the twiddles and flags, and 256 threads: four
// workgroups per compute unit (160 KB), whose barriers are independent.
constexpr int kRegN = 4096, kRegT = 256;
constexpr int kRegBuf = 4352;  // exchange buffer (elements): 256 x 17 and 16 x 272

// v exp(SIGN 2 pi i q / S) for constants S in {1, 2, 4} and q.
template <int S, int Q, int SIGN>
__device__ __forceinline__ cpx<float> turn_const(cpx<float> v) {
  constexpr int q = ((Q * (4 / S)) & 3) * (SIGN > 0 ? 1 : 3) & 3;
  if constexpr (q == 0) return v;
  if constexpr (q == 1) return {-v.y, v.x};
  if constexpr (q == 2) return {-v.x, -v.y};
  return {v.y, -v.x};
}

// exp(SIGN 2 pi i K / 64), K = 0..3
template <int K, int SIGN>
__device__ __forceinline__ cpx<float> root64() {
  static_assert(K >= 0 && K < 4, "first-stage twiddles");
  constexpr double c[4] = {1.0, 0.99518472667219688624, 0.98078528040323044913,
                           0.95694033573220886494};
  constexpr double sn[4] = {0.0, 0.09801714032956060199, 0.19509032201612826785,
                            0.29028467725446236764};
  return {(float)c[K], SIGN > 0 ? (float)sn[K] : (float)-sn[K]};
}

// Residue s: y[k3] = X[S (t + 256 k3) + s], k3 < 4 or k3 >= 12 (the central
// frequencies), from the inputs x[r] of slots t + 256 r.  buf is free on entry (every earlier read of it behind a
// barrier); its last reads, of residue s, are not followed by one.
template <int S, int s, int SIGN>
__device__ __forceinline__ void reg_fft(const cpx<float> (&x)[16], cpx<float> (&y)[16],
                                        cpx<float>* __restrict__ buf,
                                        const cpx<float>* __restrict__ tws) {
  constexpr int M = kRegN * S;
  const int t = (int)threadIdx.x, lo = t & 15, hi = t >> 4;
#pragma unroll
  for (int r = 0; r < 16; ++r)
    y[r] = r < 8 ? turn_const<S, s*(S / 2), SIGN>(x[r])
                 : turn_const<S, s*(S > 1 ? S / 2 - 1 : 0), SIGN>(x[r]);
  if constexpr (s == 0)
    dft<float, 16, SIGN>(y);
  else
    dft_tw<float, 16, SIGN>(y, root64<s * 4 / S, SIGN>());
#pragma unroll
  for (int k = 0; k < 16; ++k) buf[17 * t + k] = y[k];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = buf[17 * (hi + 16 * r) + lo];
  {
    cpx<float> u = twiddle<float, M>(tws, 16 * (S * lo + s));
    if (SIGN < 0) u.y = -u.y;
    dft_tw<float, 16, SIGN>(y, u);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) buf[272 * hi + lo + 16 * k] = y[k];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = buf[272 * r + t];
  {
    cpx<float> u = twiddle<float, M>(tws, S * t + s);
    if (SIGN < 0) u.y = -u.y;
    dft_tw<float, 16, SIGN>(y, u);
  }
  // (the central outputs are formed here, not sunk into the caller's
  // conditional stores with all their inputs alive until then)
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (k < 4 || k >= 12) asm volatile("" : "+v"(y[k].x), "+v"(y[k].y));
}

// exp(SIGN 2 pi i K / 64), any K >= 0
template <int K, int SIGN>
__device__ __forceinline__ cpx<float> root64_any() {
  constexpr double c[17] = {1.0, 0.99518472667219688624, 0.98078528040323044913,
                            0.95694033573220886494, 0.92387953251128675613,
                            0.88192126434835502971, 0.83146961230254523708,
                            0.77301045336273696081, 0.70710678118654752440,
                            0.63439328416364549822, 0.55557023301960222474,
                            0.47139673682599764856, 0.38268343236508977173,
                            0.29028467725446236764, 0.19509032201612826785,
                            0.09801714032956060199, 0.0};
  constexpr int q = K & 63, h = q >> 4, r = q & 15;
  constexpr double a = c[r], b = c[16 - r];  // cos, sin of the angle within its quadrant
  constexpr double x = h == 0 ? a : (h == 1 ? -b : (h == 2 ? -a : b));
  constexpr double y = h == 0 ? b : (h == 1 ? a : (h == 2 ? -b : -a));
  return {(float)x, (float)(SIGN > 0 ? y : -y)};
}

// The transposed transform: input on the n = 2048 S central frequencies
// c = S k + s of a length-M sequence, outputs in the window of 4096 slots
// centred on M / 2.  X[f] = sum_s w^(s f) Y_s[f mod 4096], Y_s the 4096-point
// transform of residue s, whose input holds k = t + 256 r (mod 4096) for
// r < 4 and r >= 12: thread t passes x[q] of k + 1024 = t + 256 q, q < 8.
// Adds residue s into acc[k3], the output of slot t + 256 k3.
template <int SIGN>
__device__ __forceinline__ void dft16_central(const cpx<float> (&x)[8], cpx<float> (&y)[16]) {
  // inputs r = 0..3 are x[4..7], r = 12..15 x[0..3], the others zero: one
  // decimation step leaves two 8-point transforms
  cpx<float> p[8], m[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const cpx<float> v = i < 4 ? x[i + 4] : x[i - 4];
    p[i] = v;
    m[i] = rot<float, 16, SIGN>(i < 4 ? v : cpx<float>{-v.x, -v.y}, i);
  }
  dft<float, 8, SIGN>(p);
  dft<float, 8, SIGN>(m);
#pragma unroll
  for (int f = 0; f < 8; ++f) {
    y[2 * f] = p[f];
    y[2 * f + 1] = m[f];
  }
}

template <int S, int s, int SIGN, int K3>
__device__ __forceinline__ void reg_accumulate(cpx<float> (&acc)[16], const cpx<float> (&y)[16],
                                               cpx<float> u) {
  if constexpr (K3 < 16) {
    if constexpr (s == 0) {
      acc[K3] = y[K3];
    } else {
      // w^(s f): f = t + 256 k3 + 4096 m, m = S / 2 at or above M / 2, else one less
      constexpr int m = K3 < 8 ? S / 2 : S / 2 - 1;
      const cpx<float> w = cmul(u, root64_any<(4 * s / S) * K3 + 64 * s * m / S, SIGN>());
      acc[K3].x = fmar(-w.y, y[K3].y, fmar(w.x, y[K3].x, acc[K3].x));
      acc[K3].y = fmar(w.y, y[K3].x, fmar(w.x, y[K3].y, acc[K3].y));
    }
    reg_accumulate<S, s, SIGN, K3 + 1>(acc, y, u);
  }
}

template <int S, int s, int SIGN>
__device__ __forceinline__ void reg_fft_central(const cpx<float> (&x)[8], cpx<float> (&acc)[16],
                                                cpx<float>* __restrict__ buf,
                                                const cpx<float>* __restrict__ tws) {
  constexpr int M = kRegN * S;
  const int t = (int)threadIdx.x, lo = t & 15, hi = t >> 4;
  cpx<float> y[16];
  auto tw = [&](int k) {
    cpx<float> u = twiddle<float, M>(tws, k);
    if (SIGN < 0) u.y = -u.y;
    return u;
  };
  dft16_central<SIGN>(x, y);
#pragma unroll
  for (int k = 0; k < 16; ++k) buf[17 * t + k] = y[k];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = buf[17 * (hi + 16 * r) + lo];
  dft_tw<float, 16, SIGN>(y, tw(16 * S * lo));
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) buf[272 * hi + lo + 16 * k] = y[k];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = buf[272 * r + t];
  dft_tw<float, 16, SIGN>(y, tw(S * t));
  reg_accumulate<S, s, SIGN, 0>(acc, y, s == 0 ? cpx<float>{1.f, 0.f} : tw(s * t));
  // (the sums are formed here, not sunk into a caller's conditional stores with
  // every residue's outputs alive until then)
#pragma unroll
  for (int k = 0; k < 16; ++k) asm volatile("" : "+v"(acc[k].x), "+v"(acc[k].y));
}

}  // namespace pc
