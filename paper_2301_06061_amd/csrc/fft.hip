// Batched 2-D FFT of the w-planes (Eq. 2, inner integral) and the fused
// w-screen kernels (Eq. 2, outer integral).
//
// Each 1-D transform is a Stockham autosort FFT (radix 8, one radix-4 or
// radix-2 stage last; radix 16 first where a thread holds 16 points of a
// long FP32 line) held in LDS: the first stage reads HBM directly and
// the last writes HBM directly, so a transform costs one read and one write
// of its line.  Rows are transformed one per workgroup; columns in blocks of
// BC adjacent columns per workgroup (BC * 8 or 16 bytes per row segment),
// with the blocks that share a cache line placed on one XCD so that the
// partial lines are merged in that XCD's L2.  The centring
// (DC at N/2 in both domains) is a (-1)^index sign on input and output,
// valid for every N divisible by 4.  Twiddles e^{2 pi i t/N} come from
// tables computed in FP64 once per plan.
//
// Fused kernels: after the column stage, one workgroup per image row q
// transforms row q of every plane in turn and accumulates
// F_k[q][p] exp(2 pi i w_k (n_pq - 1)) in registers, so the transformed
// planes are never written back; the degridding counterpart multiplies an
// image row by each plane's conjugate screen before transforming it.  The
// planes are equispaced in w: a step from plane to plane and the phasor of
// the first one come from FP64 sincospi of phases reduced to [-1/2, 1/2]
// turn, and are applied in the path's precision.
#include "ws_kernels.h"

namespace ws {

namespace {

__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// A pointer that is the same in all lanes, as a scalar.
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint64_t hi = uniform_u32((uint32_t)(a >> 32));
  return reinterpret_cast<const T*>(hi << 32 | uniform_u32((uint32_t)a));
}

template <typename R>
__device__ __forceinline__ cplx<R> rot_i(cplx<R> a, R s) {
  // a * (s i)
  return {-s * a.im, s * a.re};
}

template <typename R>
__device__ __forceinline__ void dft2(cplx<R>* v) {
  const cplx<R> a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <typename R>
__device__ __forceinline__ void dft4(cplx<R>* v, R s) {
  const cplx<R> a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
  const cplx<R> a2 = cadd(v[1], v[3]);
  const cplx<R> a3 = rot_i(csub(v[1], v[3]), s);
  v[0] = cadd(a0, a2);
  v[2] = csub(a0, a2);
  v[1] = cadd(a1, a3);
  v[3] = csub(a1, a3);
}

template <typename R>
__device__ __forceinline__ void dft8(cplx<R>* v, R s) {
  // Two length-4 transforms of the even and odd samples, then one radix-2
  // stage with the eighth roots of unity e^{s 2 pi i t/8}.
  cplx<R> e[4] = {v[0], v[2], v[4], v[6]};
  cplx<R> o[4] = {v[1], v[3], v[5], v[7]};
  dft4(e, s);
  dft4(o, s);
  const R h = (R)0.70710678118654752440084436210484903928;
  const cplx<R> o1 = {h * (o[1].re - s * o[1].im), h * (o[1].im + s * o[1].re)};
  const cplx<R> o2 = rot_i(o[2], s);
  const cplx<R> o3 = {h * (-o[3].re - s * o[3].im), h * (s * o[3].re - o[3].im)};
  v[0] = cadd(e[0], o[0]);
  v[4] = csub(e[0], o[0]);
  v[1] = cadd(e[1], o1);
  v[5] = csub(e[1], o1);
  v[2] = cadd(e[2], o2);
  v[6] = csub(e[2], o2);
  v[3] = cadd(e[3], o3);
  v[7] = csub(e[3], o3);
}

template <typename R>
__device__ __forceinline__ void dft16(cplx<R>* v, R s) {
  // n = 4 n1 + n2, k = k1 + 4 k2: length-4 transforms over n1, the twiddles
  // W16^(n2 k1), length-4 transforms over n2.
  const R h = (R)0.70710678118654752440084436210484903928;
  const R c = (R)0.92387953251128675612818318939678828682;  // cos(pi / 8)
  const R d = (R)0.38268343236508977172845998403039886676;  // sin(pi / 8)
  cplx<R> y[4][4];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    cplx<R> t[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
    dft4(t, s);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) y[k1][n2] = t[k1];
  }
  auto w2 = [&](cplx<R> a) -> cplx<R> {  // times e^{s 2 pi i 2/16}
    return {h * (a.re - s * a.im), h * (a.im + s * a.re)};
  };
  auto w6 = [&](cplx<R> a) -> cplx<R> {  // times e^{s 2 pi i 6/16}
    return {h * (-a.re - s * a.im), h * (s * a.re - a.im)};
  };
  y[1][1] = cmul(y[1][1], cplx<R>{c, s * d});
  y[1][2] = w2(y[1][2]);
  y[1][3] = cmul(y[1][3], cplx<R>{d, s * c});
  y[2][1] = w2(y[2][1]);
  y[2][2] = rot_i(y[2][2], s);
  y[2][3] = w6(y[2][3]);
  y[3][1] = cmul(y[3][1], cplx<R>{d, s * c});
  y[3][2] = w6(y[3][2]);
  y[3][3] = cmul(y[3][3], cplx<R>{-c, -s * d});
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    dft4(y[k1], s);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = y[k1][k2];
  }
}

template <typename R, int RAD>
__device__ __forceinline__ void dft(cplx<R>* v, R s) {
  if constexpr (RAD == 16) dft16(v, s);
  else if constexpr (RAD == 8) dft8(v, s);
  else if constexpr (RAD == 4) dft4(v, s);
  else dft2(v);
}

// Twiddles e^{s 2 pi i idx/N} from two small LDS tables, e^{2 pi i lo/N}
// for lo < 64 and e^{2 pi i 64 hi/N}, both rounded from FP64 values.
template <typename R>
struct Twiddles {
  const cplx<R>* t_lo;
  const cplx<R>* t_hi;
  __device__ __forceinline__ cplx<R> operator()(int idx, R s) const {
    const cplx<R> a = t_lo[idx & 63], b = t_hi[idx >> 6];
    const cplx<R> w = cmul(a, b);
    return {w.re, s * w.im};
  }
  // w[i] = W^(i k N / (NS RAD)), i = 1, 2, 4, 8 < RAD, of stage P: lookups
  // of i = 1 and, for radix 16, i = 4; the others as squares (a few units in
  // the last place).
  static constexpr bool kAll = false;
  template <int LOGN, bool WIDE, int P, int RAD, int NS>
  __device__ __forceinline__ void stage(int k, int, R s, cplx<R>* w) const {
    constexpr int step = (1 << LOGN) / (NS * RAD);
    w[1] = (*this)(k * step, s);
    if constexpr (RAD > 2) w[2] = cmul(w[1], w[1]);
    if constexpr (RAD == 8) w[4] = cmul(w[2], w[2]);
    if constexpr (RAD == 16) {
      w[4] = (*this)(4 * k * step, s);
      w[8] = cmul(w[4], w[4]);
    }
  }
};

constexpr int kTwLo = 64;

// Fill the LDS twiddle tables of a length-n transform from the global table.
template <typename R>
__device__ __forceinline__ Twiddles<R> load_twiddles(cplx<R>* s_lo,
                                                     cplx<R>* s_hi,
                                                     const cplx<R>* tw, int n) {
  for (int i = threadIdx.x; i < kTwLo; i += blockDim.x) s_lo[i] = tw[i % n];
  for (int i = threadIdx.x; i < (n + kTwLo - 1) / kTwLo; i += blockDim.x)
    s_hi[i] = tw[i * kTwLo];
  return Twiddles<R>{s_lo, s_hi};
}

// Tables of a length-n sub-transform inside a length-nfull table
// (W_n^x = W_nfull^(x * nfull / n)), for the two steps of a four-step
// transform.
template <typename R>
__device__ __forceinline__ Twiddles<R> load_twiddles_sub(cplx<R>* s_lo,
                                                         cplx<R>* s_hi,
                                                         const cplx<R>* tw,
                                                         int n, int nfull) {
  const int stride = nfull / n;
  for (int i = threadIdx.x; i < kTwLo; i += blockDim.x)
    s_lo[i] = tw[((i % n) * stride) & (nfull - 1)];
  for (int i = threadIdx.x; i < (n + kTwLo - 1) / kTwLo; i += blockDim.x)
    s_hi[i] = tw[(i * kTwLo * stride) & (nfull - 1)];
  return Twiddles<R>{s_lo, s_hi};
}

// LDS slot of line element e: one padding slot after every 32 elements,
// so that the strided accesses of the Stockham stages spread over the
// banks (measured against one slot per 8, 16 and 64 elements: the fewest
// bank conflicts and the fastest column and row passes).
__device__ __forceinline__ constexpr int lslot(int e) { return e + (e >> 5); }

template <int N>
constexpr int lds_line(int bc) {
  return (N + (N + 31) / 32) * bc;
}

// Pass structure of a length-2^LOGN transform, as bits per stage: radix 8 and
// the remainder (radix 2 or 4) last; or, WIDE (LOGN >= 10), radix 16 first
// and radix 8 after, as few stages as possible.  Every stage but the first
// costs a write and a read of the line in LDS, which is what bounds these
// kernels (measured per CU and wavefront instruction: 8-byte LDS write 7.1
// cycles, read 4.4, FP32 fma 0.7): 16 x 16 x 16 exchanges a 4096-point line
// twice, 8 x 8 x 8 x 8 three times.  WIDE needs 16 elements a thread.
constexpr bool plan_wide(int logn, bool wide) { return wide && logn >= 10; }
constexpr int stage_bits(int logn, bool wide, int P) {
  if (plan_wide(logn, wide)) return P < (logn - 10) % 3 + 1 ? 4 : 3;
  return P < logn / 3 ? 3 : logn % 3;
}
constexpr int stage_log_ns(int logn, bool wide, int P) {
  int b = 0;
  for (int q = 0; q < P; ++q) b += stage_bits(logn, wide, q);
  return b;
}
constexpr int stage_npass(int logn, bool wide) {
  int P = 0;
  while (stage_log_ns(logn, wide, P) < logn) ++P;
  return P;
}
// Offset of stage P's entries in a stage twiddle table (stages 1 ..).
constexpr int stage_tw_off(int logn, bool wide, int P) {
  int o = 0;
  for (int q = 1; q < P; ++q)
    o += stage_bits(logn, wide, q) << stage_log_ns(logn, wide, q);
  return o;
}
constexpr int stage_tw_total(int logn, bool wide) {
  return stage_tw_off(logn, wide, stage_npass(logn, wide));
}

// Twiddles of every stage in LDS: stage P keeps W^(i k N / (NS RAD)) for i =
// 1, 2, 4, (8) < RAD and k < NS at tab[stage_tw_off(P) + log2(i) NS + k]
// (lanes read consecutive k), the transform sign applied when the table is
// filled; the other powers are one or two products of these.
template <typename R>
struct TableTwiddles {
  static constexpr bool kAll = false;
  const cplx<R>* tab;
  template <int LOGN, bool WIDE, int P, int RAD, int NS>
  __device__ __forceinline__ void stage(int k, int, R, cplx<R>* w) const {
    constexpr int OFF = stage_tw_off(LOGN, WIDE, P);
    w[1] = tab[OFF + k];
    if constexpr (RAD > 2) w[2] = tab[OFF + NS + k];
    if constexpr (RAD > 4) w[4] = tab[OFF + 2 * NS + k];
    if constexpr (RAD > 8) w[8] = tab[OFF + 3 * NS + k];
  }
};

// Fills the stage table of a length-2^LOGN transform from the global table
// tw of a length-(stride 2^LOGN) one, conjugated for s = -1.
template <typename R, int LOGN, bool WIDE>
__device__ __forceinline__ void fill_stage_twiddles(cplx<R>* tab,
                                                    const cplx<R>* tw, R s,
                                                    int stride) {
  constexpr int N = 1 << LOGN;
  constexpr int NPASS = stage_npass(LOGN, WIDE);
  for (int i = threadIdx.x; i < stage_tw_total(LOGN, WIDE); i += blockDim.x) {
    int idx = 0;
#pragma unroll
    for (int P = 1; P < NPASS; ++P) {
      const int off = stage_tw_off(LOGN, WIDE, P);
      const int lns = stage_log_ns(LOGN, WIDE, P);
      const int bits = stage_bits(LOGN, WIDE, P);
      if (i >= off && i < off + (bits << lns)) {
        const int l = (i - off) >> lns, k = (i - off) & ((1 << lns) - 1);
        idx = ((k << l) << (LOGN - lns - bits)) & (N - 1);
      }
    }
    const cplx<R> w = tw[(size_t)idx * stride];
    tab[i] = {w.re, s * w.im};
  }
}

// Row twiddles: every factor W^(r k N / (NS RAD)), r = 1 .. RAD-1, as the
// plan's table has it, rounded once (factors formed as products of others
// carry one or two roundings more: 12-18% on the error of a row transform).
// The stages in the middle read theirs from LDS, FP32 factors in pairs (r =
// 1 and 2, 3 and 4, ...: one 16-byte read each).  The last stage's are most
// of a full table (28 of 32 KB at 4096 FP32 points), and a thread meets the
// same ones on every plane: they stay in its registers, but for the first LF
// where LDS has room and registers are short.  Row pass of 32 planes of
// 4096^2 (FP32 / FP64) and 16 of 2048^2 (FP32), us: factors 1, 2, 4 and
// products of them 953 / 1970 / 124; these 947 / 1947 / 120; with LF = 0 at
// 4096 1105 / 2030 (spills); LF = 3 at 2048, which leaves no room for the
// seeds in LDS, 128.
template <typename R, int LOGN, int NT>
struct RowTwiddles {
  static constexpr bool kAll = true;
  static constexpr int N = 1 << LOGN;
  static constexpr int LAST = stage_npass(LOGN, false) - 1;
  static constexpr int RAD = 1 << stage_bits(LOGN, false, LAST);
  static constexpr int NS = N / RAD;
  static constexpr int IT = (NS + NT - 1) / NT;
  static constexpr int LF =
      LOGN == 12 ? 2 : (sizeof(R) == 4 && LOGN == 10 ? RAD - 1 : 0);
  static constexpr bool PAIRS = sizeof(R) == 4;
  // Factors of stage P in LDS, and the first entry of the stage's.
  static constexpr int factors(int P) {
    return P == LAST ? LF : (1 << stage_bits(LOGN, false, P)) - 1;
  }
  static constexpr int off(int P) {
    int o = 0;
    for (int q = 1; q < P; ++q)
      o += factors(q) << stage_log_ns(LOGN, false, q);
    return o;
  }
  static constexpr int kTab = off(LAST) + LF * NS;
  const cplx<R>* tab;  // 16-byte aligned
  cplx<R> last[IT][RAD];

  // Fills s_tab (kTab entries) and this thread's last stage from the plan's
  // table, conjugated for s = -1.  The last stage's also carry the input
  // centring: a (-1)^e factor of the input gives every butterfly of the
  // earlier stages one common sign, which the Stockham order carries to input
  // r of the last stage as (-1)^r.
  __device__ __forceinline__ RowTwiddles(cplx<R>* s_tab, const cplx<R>* tw,
                                         R s, int tid)
      : tab(s_tab) {
    auto entry = [&](int idx, bool neg) -> cplx<R> {
      const cplx<R> w = tw[idx];
      return neg ? cplx<R>{-w.re, -s * w.im} : cplx<R>{w.re, s * w.im};
    };
    for (int i = threadIdx.x; i < kTab; i += blockDim.x) {
      int idx = 0;
      bool neg = false;
#pragma unroll
      for (int P = 1; P <= LAST; ++P) {
        const int lns = stage_log_ns(LOGN, false, P);
        const int bits = stage_bits(LOGN, false, P);
        const int j = i - off(P), nf = factors(P);
        if (j < 0 || j >= nf << lns) continue;
        int r = (j >> lns) + 1, k = j & ((1 << lns) - 1);
        if (PAIRS && ((r - 1) | 1) < nf) {
          const int h = j & ((2 << lns) - 1);
          r = (j >> (lns + 1)) * 2 + (h & 1) + 1;
          k = h >> 1;
        }
        idx = (r * k) << (LOGN - lns - bits);
        neg = P == LAST && (r & 1);
      }
      s_tab[i] = entry(idx, neg);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int k = (tid + it * NT) & (NS - 1);
#pragma unroll
      for (int r = 1 + LF; r < RAD; ++r) last[it][r] = entry(r * k, r & 1);
    }
  }
  template <int, bool, int P, int SRAD, int SNS>
  __device__ __forceinline__ void stage(int k, int it, R, cplx<R>* w) const {
    constexpr int NF = factors(P);
    const cplx<R>* t = tab + off(P);
#pragma unroll
    for (int r = 1; r < SRAD; ++r) {
      if (r > NF) {
        w[r] = last[it][r];
      } else if (PAIRS && ((r - 1) | 1) < NF) {
        if (r & 1) {
          struct alignas(2 * sizeof(cplx<R>)) Pair { cplx<R> a, b; };
          const Pair p =
              reinterpret_cast<const Pair*>(t + (r - 1) * SNS)[k];
          w[r] = p.a;
          w[r + 1] = p.b;
        }
      } else {
        w[r] = t[(r - 1) * SNS + k];
      }
    }
  }
};

// Inputs r = 1 .. RAD-1 of a butterfly times w[r], given whole (ALL) or as
// w[1], w[2], w[4], w[8].
template <typename R, int RAD, bool ALL>
__device__ __forceinline__ void apply_twiddles(cplx<R>* v, cplx<R>* w) {
  if constexpr (!ALL) {
#pragma unroll
    for (int i = 1; i < RAD; i *= 2) {
#pragma unroll
      for (int r = i + 1; r < 2 * i; ++r) w[r] = cmul(w[r - i], w[i]);
    }
  }
#pragma unroll
  for (int r = 1; r < RAD; ++r) v[r] = cmul(v[r], w[r]);
}

// Stage P of a length-2^LOGN Stockham FFT over BC interleaved columns
// (element e of column c at lds[e * BC + c]).  Stage 0 reads through
// ld(e, c); the last stage hands each output to st(e, c, it, r, value).
template <typename R, int LOGN, int BC, int NT, int P, bool WIDE = false>
struct Stage {
  static constexpr int N = 1 << LOGN;
  static constexpr int NPASS = stage_npass(LOGN, WIDE);
  static constexpr int RAD = 1 << stage_bits(LOGN, WIDE, P);
  static constexpr int NS = 1 << stage_log_ns(LOGN, WIDE, P);
  static constexpr int NB = N / RAD;
  static constexpr int TPC = NT / BC;
  static constexpr int IT = (NB + TPC - 1) / TPC;
  static constexpr bool FIRST = P == 0;
  static constexpr bool LAST = P == NPASS - 1;

  template <class Load, class Store, class TW>
  __device__ __forceinline__ static void run(cplx<R>* lds, const Load& ld,
                                             const Store& st, const TW& tw,
                                             R s, int tid) {
    const int c = tid % BC;
    const int jt = tid / BC;
    cplx<R> v[IT][RAD];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int j = jt + it * TPC;
      if (NB % TPC == 0 || j < NB) {
#pragma unroll
        for (int r = 0; r < RAD; ++r) {
          const int e = j + r * NB;
          if constexpr (FIRST) v[it][r] = ld(e, c, it, r);
          else v[it][r] = lds[lslot(e) * BC + c];
        }
      }
    }
    if constexpr (!FIRST) __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int j = jt + it * TPC;
      if (NB % TPC == 0 || j < NB) {
        const int k = j & (NS - 1);
        if constexpr (NS > 1) {
          // Twiddles W^(r k N / (NS RAD)), r = 1 .. RAD-1.
          cplx<R> w[RAD];
          tw.template stage<LOGN, WIDE, P, RAD, NS>(k, it, s, w);
          apply_twiddles<R, RAD, TW::kAll>(v[it], w);
        }
        dft<R, RAD>(v[it], s);
        if constexpr (LAST) {
#pragma unroll
          for (int r = 0; r < RAD; ++r) st(j + r * NB, c, it, r, v[it][r]);
        } else {
          const int ob = (j / NS) * NS * RAD + k;
#pragma unroll
          for (int r = 0; r < RAD; ++r)
            lds[lslot(ob + r * NS) * BC + c] = v[it][r];
        }
      }
    }
    if constexpr (!LAST) {
      __syncthreads();
      Stage<R, LOGN, BC, NT, P + 1, WIDE>::run(lds, ld, st, tw, s, tid);
    }
  }
};

// NT threads (tid = 0 .. NT-1 within the line's group; every group of the
// workgroup calls together) transform one line, or BC interleaved columns.
template <typename R, int LOGN, int BC, int NT, bool WIDE = false, class Load,
          class Store, class TW>
__device__ __forceinline__ void fft_line(cplx<R>* lds, const Load& ld,
                                         const Store& st, const TW& tw, R s,
                                         int tid) {
  Stage<R, LOGN, BC, NT, 0, WIDE>::run(lds, ld, st, tw, s, tid);
}

template <typename R, int LOGN, int BC, int NT, bool WIDE = false, class Load,
          class Store, class TW>
__device__ __forceinline__ void fft_line(cplx<R>* lds, const Load& ld,
                                         const Store& st, const TW& tw, R s) {
  Stage<R, LOGN, BC, NT, 0, WIDE>::run(lds, ld, st, tw, s, (int)threadIdx.x);
}

template <typename R>
__device__ __forceinline__ cplx<R> checker(cplx<R> v, int e) {
  return (e & 1) ? cplx<R>{-v.re, -v.im} : v;
}

// ---- plain row and column transforms (in place, any plane count) --------

// Sample e of a stack row whose 64-column strips carry marks (mk: the
// plane's marks, null when every strip holds data): read where the strip
// is marked, zero elsewhere (the load then goes to the spare line, so it
// costs no HBM traffic and needs no branch).  e - threadIdx.x must be the
// same across the workgroup and a multiple of 64, as in the first-stage
// loads of the row transforms, so that a wavefront's 64 samples lie in one
// strip and every choice here is wavefront-uniform.
template <bool MK, typename R>
__device__ __forceinline__ cplx<R> row_sample(const cplx<R>* line, int e,
                                              const uint32_t* __restrict__ mk,
                                              const cplx<R>* spare) {
  if constexpr (!MK) return line[e];
  const int c = e - (int)threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const bool on = mk[w + (c >> 6)] != 0u;
  const char* sb = on ? reinterpret_cast<const char*>(line + c)
                      : reinterpret_cast<const char*>(spare);
  const cplx<R> v = *reinterpret_cast<const cplx<R>*>(
      sb + (size_t)threadIdx.x * sizeof(cplx<R>));
  return cplx<R>{on ? v.re : (R)0, on ? v.im : (R)0};
}

// Marks of the plane that stack row `row` belongs to (null: no marks).
__device__ __forceinline__ const uint32_t* row_marks(const uint32_t* strips,
                                                     int64_t row,
                                                     int rows_per_plane,
                                                     int strips_per_row) {
  return strips == nullptr
             ? nullptr
             : strips + (size_t)(row / rows_per_plane) * strips_per_row;
}

// MK: with `strips` (marks of the 64-column strips of each plane of
// rows_per_plane rows), samples of unmarked strips are taken as zero and
// not read: the one-call path leaves those strips unwritten.
template <typename R, int LOGN, int NT, bool MK>
__global__ __launch_bounds__(NT) void k_fft_rows(
    cplx<R>* data, int64_t nrows, const cplx<R>* __restrict__ tw, R s,
    const uint32_t* __restrict__ strips, int rows_per_plane,
    int strips_per_row) {
  constexpr int N = 1 << LOGN;
  __shared__ cplx<R> lds[lds_line<N>(1)];
  __shared__ cplx<R> s_lo[kTwLo], s_hi[(N + kTwLo - 1) / kTwLo];
  const int64_t row = blockIdx.x;
  if (row >= nrows) return;
  const Twiddles<R> twl = load_twiddles(s_lo, s_hi, tw, N);
  __syncthreads();
  cplx<R>* line = data + row * N;
  static_assert(!MK || (NT % 64 == 0 && (N / 8) % 64 == 0),
                "marks need one strip per wavefront");
  const uint32_t* mk =
      MK ? row_marks(strips, row, rows_per_plane, strips_per_row) : nullptr;
  auto ld = [&](int e, int, int, int) {
    return checker(row_sample<MK>(line, e, mk, tw), e);
  };
  auto st = [&](int e, int, int, int, cplx<R> v) { line[e] = checker(v, e); };
  fft_line<R, LOGN, 1, NT>(lds, ld, st, twl, s);
}

template <typename R>
__device__ __forceinline__ cplx<R> twiddle_full(const cplx<R>* tw, int idx,
                                                R s) {
  const cplx<R> w = tw[idx];
  return {w.re, s * w.im};
}

// Rows too long for one workgroup's LDS (2N elements of FP64 at N = 16384):
// one radix-2 decimation-in-frequency step in registers, then two LDS
// transforms of half length.  With x' = (-1)^n x (centring),
//   X[2k]   = DFT_{N/2}( x'[n] + x'[n + N/2] )
//   X[2k+1] = DFT_{N/2}( (x'[n] - x'[n + N/2]) W_N^n ).
// Both halves of the row are read once (coalesced); the difference terms
// wait in registers while the sum terms are transformed, and the two
// outputs of each k are written together.
template <typename R, int LOGH, int NT, bool MK>
__global__ __launch_bounds__(NT) void k_fft_rows_split(
    cplx<R>* data, int64_t nrows, const cplx<R>* __restrict__ tw, R s,
    const uint32_t* __restrict__ strips, int rows_per_plane,
    int strips_per_row) {
  constexpr int NH = 1 << LOGH;  // half length
  constexpr int N = 2 * NH;
  __shared__ cplx<R> lds[lds_line<NH>(1)];
  __shared__ cplx<R> s_lo[kTwLo], s_hi[(NH + kTwLo - 1) / kTwLo];
  using F0 = Stage<R, LOGH, 1, NT, 0>;
  using FL = Stage<R, LOGH, 1, NT, F0::NPASS - 1>;
  const int64_t row = blockIdx.x;
  if (row >= nrows) return;
  cplx<R>* line = data + row * N;
  const Twiddles<R> twl = load_twiddles_sub(s_lo, s_hi, tw, NH, N);
  __syncthreads();
  cplx<R> diff[F0::IT][F0::RAD];
  cplx<R> even[FL::IT][FL::RAD];
  static_assert(!MK || (NT % 64 == 0 && F0::NB % 64 == 0 && NH % 64 == 0),
                "marks need one strip per wavefront");
  const uint32_t* mk =
      MK ? row_marks(strips, row, rows_per_plane, strips_per_row) : nullptr;
  auto ld_sum = [&](int e, int, int it, int r) {
    const cplx<R> a = checker(row_sample<MK>(line, e, mk, tw), e);
    const cplx<R> b = checker(row_sample<MK>(line, e + NH, mk, tw), e + NH);
    diff[it][r] = cmul(csub(a, b), twiddle_full(tw, e, s));
    return cadd(a, b);
  };
  auto st_even = [&](int, int, int it, int r, cplx<R> v) { even[it][r] = v; };
  fft_line<R, LOGH, 1, NT>(lds, ld_sum, st_even, twl, s);
  auto ld_diff = [&](int, int, int it, int r) { return diff[it][r]; };
  auto st_odd = [&](int e, int, int it, int r, cplx<R> v) {
    // output 2e is even (sign +1), 2e + 1 is odd (sign -1)
    const cplx<R> lo = even[it][r];
    const cplx<R> hi = {-v.re, -v.im};
    line[2 * e] = lo;
    line[2 * e + 1] = hi;
  };
  fft_line<R, LOGH, 1, NT>(lds, ld_diff, st_odd, twl, s);
}

// Rows too long even for two half-length LDS transforms (FP64 at 32768):
// F-way decimation in frequency with F = 4.  With x' = (-1)^n x and
// NF = N / F,
//   X[F k + r] = DFT_NF( W_N^(s r n) sum_m x'[n + m NF] W_F^(s m r) )[k],
// so output class r is one length-NF transform of a combination of the F
// samples x'[n + m NF]; output F k + r carries the centring sign (-1)^r.
// Pass r re-reads the row (F samples per point) instead of keeping the
// other classes in registers (at FP64 they would need ~200 registers a
// thread), and writes its outputs to the workgroup's row of `scratch`
// (every class reads the whole row, so nothing can be written in place
// before the last class); the finished row is then copied back.
// Persistent: workgroup b transforms rows b, b + G, ... (G = grid size),
// with scratch rows [G][N].  Only for grids wider than the fused kernels
// handle.
template <typename R, int LOGF, int NT, int F>
__global__ __launch_bounds__(NT) void k_fft_rows_splitF(
    cplx<R>* data, int64_t nrows, const cplx<R>* __restrict__ tw, R s,
    cplx<R>* __restrict__ scratch) {
  constexpr int NF = 1 << LOGF;
  constexpr int N = F * NF;
  __shared__ cplx<R> lds[lds_line<NF>(1)];
  __shared__ cplx<R> s_lo[kTwLo], s_hi[(NF + kTwLo - 1) / kTwLo];
  const Twiddles<R> twl = load_twiddles_sub(s_lo, s_hi, tw, NF, N);
  __syncthreads();
  cplx<R>* tmp = scratch + (size_t)blockIdx.x * N;
  for (int64_t row = blockIdx.x; row < nrows; row += gridDim.x) {
    cplx<R>* line = data + row * N;
    for (int r = 0; r < F; ++r) {
      auto ld = [&](int e, int, int, int) {
        cplx<R> acc = {(R)0, (R)0};
#pragma unroll
        for (int m = 0; m < F; ++m) {
          const int idx = e + m * NF;
          const cplx<R> x = checker(line[idx], idx);
          acc = cadd(acc,
                     cmul(x, twiddle_full(tw, (m * r * NF) & (N - 1), s)));
        }
        return cmul(acc, twiddle_full(tw, (r * e) & (N - 1), s));
      };
      const R sg = (r & 1) ? (R)-1 : (R)1;
      auto st = [&](int e, int, int, int, cplx<R> v) {
        tmp[F * e + r] = cplx<R>{sg * v.re, sg * v.im};
      };
      fft_line<R, LOGF, 1, NT>(lds, ld, st, twl, s);
      __syncthreads();
    }
    // Scratch row complete (global writes of this workgroup, ordered by
    // the barrier's release / acquire at workgroup scope): copy it back.
    __threadfence_block();
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += NT) line[i] = tmp[i];
    __syncthreads();
  }
}

// Workgroups of k_fft_rows_splitF (and scratch rows it needs).
constexpr int kSplitRowGroups = 256;

// Which rows of a column block hold data, from the per-tile record
// counts of gridding (0 = a tile without records, whose cells a fused
// grid-and-image call leaves unwritten and the transform takes as zero).
// The counts of the block's tile column (at most 64 tile rows) become one
// 64-bit mask per wavefront in the prologue, so every element then costs a
// shift and a select: no load, no branch, and the data loads of a
// wavefront still issue back to back.  Without a table every row holds
// data.
struct TileRows {
  unsigned long long mask;
  int log_t;
  // Issues the load of this lane's tile count (without a table, of any
  // valid word `any`, then ignored: the load stays unconditional and
  // nothing waits for it here); finish() turns the counts into the mask,
  // so other loads can be issued in between.
  __device__ __forceinline__ TileRows(const uint32_t* tiles, int plane,
                                      int nrows, int ncols, int col0,
                                      int log_t_, const void* any)
      : mask(~0ull), log_t(log_t_), rows(nrows >> log_t_),
        table(tiles != nullptr) {
    const int tw = ncols >> log_t;
    const int lane = (int)(threadIdx.x & 63);
    const uint32_t* src =
        table ? tiles + (size_t)plane * rows * tw + (col0 >> log_t) +
                    (size_t)min(lane, rows - 1) * tw
              : (const uint32_t*)any;
    count = *src;
  }
  __device__ __forceinline__ void finish() {
    const unsigned long long m =
        __ballot((int)(threadIdx.x & 63) < rows && count != 0u);
    mask = table ? m : ~0ull;
  }
  __device__ __forceinline__ bool has(int e) const {
    return ((mask >> (e >> log_t)) & 1ull) != 0ull;
  }
  // Sample of row e: loaded from p where the row holds data; elsewhere the
  // load goes to `spare` (one line that every such lane shares, so it costs
  // no HBM traffic) and the value is replaced by zero.  The load itself is
  // unconditional, so a wavefront issues its loads back to back.
  template <typename R>
  __device__ __forceinline__ cplx<R> load(int e, const cplx<R>* p,
                                          const cplx<R>* spare) const {
    const bool h = has(e);
    const cplx<R> v = *(h ? p : spare);
    return cplx<R>{h ? v.re : (R)0, h ? v.im : (R)0};
  }

 private:
  uint32_t count;
  int rows;
  bool table;
};

// Logical column block of hardware block b.  Blocks are dispatched to the
// eight XCDs in turn (b % 8); the G logical blocks that share one 128-byte
// line of every row are given to one XCD (they then share its L2), and
// successive groups go to successive XCDs, so every XCD holds an equal
// share of every plane (planes can differ widely in how many of their
// column strips are skipped).  Grids that are not a multiple of 8 G blocks
// keep the identity order.
template <typename R, int BC>
__device__ __forceinline__ int xcd_block(int b, int nb) {
  constexpr int W = BC * (int)sizeof(cplx<R>);
  constexpr int G = W >= 128 ? 1 : 128 / W;
  if (nb % (8 * G) != 0) return b;
  const int x = b % 8, n = b / 8;
  return ((n / G) * 8 + x) * G + n % G;
}

template <typename R, int LOGN, int BC, int NT>
__global__ __launch_bounds__(NT) void k_fft_cols(
    cplx<R>* data, int ncols, int nplanes, const cplx<R>* __restrict__ tw, R s,
    const uint32_t* __restrict__ strips, int log_strip,
    const uint32_t* __restrict__ tiles) {
  constexpr int N = 1 << LOGN;  // column length = number of rows
  __shared__ cplx<R> lds[lds_line<N>(BC)];
  __shared__ cplx<R> s_lo[kTwLo], s_hi[(N + kTwLo - 1) / kTwLo];
  const int nb_plane = ncols / BC;
  const int nb = nb_plane * nplanes;
  const int L = xcd_block<R, BC>((int)blockIdx.x, nb);
  if (L >= nb) return;
  const int plane = L / nb_plane;
  const int col0 = (L - plane * nb_plane) * BC;
  if (strips != nullptr &&
      strips[plane * (ncols >> log_strip) + (col0 >> log_strip)] == 0u)
    return;
  cplx<R>* base = data + (size_t)plane * N * ncols + col0;
  TileRows tr(tiles, plane, N, ncols, col0, log_strip, base);
  tr.finish();
  auto ld = [&](int e, int c, int, int) {
    return checker(tr.load(e, base + (size_t)e * ncols + c, tw), e);
  };
  auto st = [&](int e, int c, int, int, cplx<R> v) {
    base[(size_t)e * ncols + c] = checker(v, e);
  };
  const Twiddles<R> twl = load_twiddles(s_lo, s_hi, tw, N);
  __syncthreads();
  fft_line<R, LOGN, BC, NT>(lds, ld, st, twl, s);
}

// Column transform with twice the columns per workgroup that a whole
// column of LDS allows: one radix-2 decimation-in-frequency step as the
// samples arrive from HBM (rows e and e + N/2), the sums transformed in
// LDS first (outputs 2e, written at once: every input has been read)
// while the twiddled differences wait in registers, then the differences
// (outputs 2e + 1).  The wider block doubles the row segment each access
// moves (64 bytes instead of 32 for 4096-point FP32 columns).
//
// TS: the input tiles are read from the busy-tile store (tstore, slot of
// tile t at tslot[t], layout tile_store_at) instead of the stack: the BC
// columns of a block are one 64-byte sub-block of each tile, so every
// tile row a wavefront reads is 512 contiguous bytes.  Tiles with a slot
// of tcap or more did not fit the store and are read from the stack.
// Needs 64-row tiles and strips, BC = 64 bytes of columns and 64 rows per
// wavefront pass (TPC = 64); the output still goes to the stack.
template <typename R, int LOGH, int BC, int NT, bool TS>
__global__ __launch_bounds__(NT) void k_fft_cols_split(
    cplx<R>* data, int ncols, int nplanes, const cplx<R>* __restrict__ tw, R s,
    const uint32_t* __restrict__ strips, int log_strip,
    const uint32_t* __restrict__ tiles, const cplx<R>* __restrict__ tstore,
    const uint32_t* __restrict__ tslot, uint32_t tcap) {
  constexpr int NH = 1 << LOGH;  // half the column length
  constexpr int N = 2 * NH;
  __shared__ cplx<R> lds[lds_line<NH>(BC)];
  // FP32: stage twiddles in a table, radix-16 stages for the longest columns
  // (one LDS exchange less); FP64 has the registers and LDS for neither.
  // 4096^2 x 32 planes of the stack, ms: FP32 2.93 -> 2.80, 2048^2 x 16
  // 0.198 -> 0.188; from the busy-tile store 1.36 -> 1.37 (not used); FP64
  // with the table 2.71 -> 2.74, with radix 16 (512 threads) 2.78.
  constexpr bool TABLE = sizeof(R) == 4 && !TS, WIDE = TABLE && LOGH == 11;
  constexpr int TAB = TABLE ? stage_tw_total(LOGH, WIDE)
                            : kTwLo + (NH + kTwLo - 1) / kTwLo;
  __shared__ cplx<R> s_tab[TAB];
  __shared__ cplx<R> f_lo[kTwLo], f_hi[N / kTwLo];
  using F0 = Stage<R, LOGH, BC, NT, 0, WIDE>;
  const int nb_plane = ncols / BC;
  const int nb = nb_plane * nplanes;
  const int L = xcd_block<R, BC>((int)blockIdx.x, nb);
  if (L >= nb) return;
  const int plane = L / nb_plane;
  const int col0 = (L - plane * nb_plane) * BC;
  if (strips != nullptr &&
      strips[plane * (ncols >> log_strip) + (col0 >> log_strip)] == 0u)
    return;
  cplx<R>* base = data + (size_t)plane * N * ncols + col0;
  // Without the stage table the prologue's loads go first (the hardware
  // returns loads in order): one entry of the four twiddle tables per thread
  // (W_NH^m and W_NH^(64 m) for the half-length stages, W_N^m and W_N^(64 m)
  // for the difference terms), then the tile counts.
  static_assert(NT >= 4 * kTwLo && N / kTwLo <= kTwLo, "one entry a thread");
  const int tq = min((int)threadIdx.x / kTwLo, 3), tm = threadIdx.x % kTwLo;
  const int tidx = tq == 0   ? 2 * tm
                   : tq == 1 ? tm
                   : tq == 2 ? 2 * kTwLo * min(tm, NH / kTwLo - 1)
                             : kTwLo * min(tm, N / kTwLo - 1);
  cplx<R> tval;
  if constexpr (!TABLE) tval = tw[tidx];
  TileRows tr(tiles, plane, N, ncols, col0, log_strip, base);
  // TS: lane l holds the store slot of tile row l of this strip (any
  // value where the tile has no records: such rows are never read).
  int myslot = 0;
  if constexpr (TS) {
    const int rows = N >> log_strip, tcols = ncols >> log_strip;
    const int lane = (int)(threadIdx.x & 63);
    myslot = (int)tslot[((size_t)plane * rows + min(lane, rows - 1)) * tcols +
                        (col0 >> log_strip)];
  }
  if constexpr (!TABLE) {
    if (threadIdx.x < 4 * kTwLo) {
      if (tq == 0) s_tab[tm] = tval;
      else if (tq == 1) f_lo[tm] = tval;
      else if (tq == 2) { if (tm < NH / kTwLo) s_tab[kTwLo + tm] = tval; }
      else if (tm < N / kTwLo) f_hi[tm] = tval;
    }
    __syncthreads();
  }
  tr.finish();
  cplx<R> diff[F0::IT][F0::RAD];
  // The first stage takes the thread's sample pairs in order n = it * RAD +
  // r; the pair n + AHEAD is requested when pair n is combined, so each
  // wavefront keeps 2 AHEAD + 2 loads in flight without holding the whole
  // strip in registers (with one workgroup per CU there is no other
  // workgroup to hide the latency).  FP32 (512 threads, 256 registers)
  // runs 4 pairs ahead from the stack and 8 from the busy-tile store;
  // FP64 at 1024 threads has no registers to spare and loads each pair
  // where it is used (measured fastest for each; requesting every pair
  // before any arithmetic measured slower for both; from the store, 2, 4,
  // 6, 12 and 16 pairs ahead measured slower than 8).
  constexpr int AHEAD = sizeof(R) == 4 ? (TS ? 8 : 4) : 0;
  constexpr int NE = F0::IT * F0::RAD;
  const int c0 = (int)threadIdx.x % BC, jt = (int)threadIdx.x / BC;
  cplx<R> qa[NE], qb[NE];
  // TS addressing: row e = jt + it TPC + r NB lies in tile row
  // (it TPC + r NB) / 64 (a constant once unrolled; jt < 64) at row jt of
  // the tile, and the block's columns are sub-block (col0 % 64) / BC.  A
  // load address is a wavefront-uniform base (the tile's slot, the row
  // in the stack for a tile past the store's last slot, or the spare line
  // for a tile without records) plus one of two per-lane byte offsets, so
  // choosing between the three costs one vector select.
  const char* ts_base = nullptr;
  uint32_t v_ts = 0, v_st = 0;
  if constexpr (TS) {
    static_assert(F0::TPC == 64 && F0::NB % 64 == 0 && NH % 64 == 0 &&
                      BC * sizeof(cplx<R>) == 64,
                  "busy-tile store: 64-row tiles, 64-byte sub-blocks");
    ts_base = reinterpret_cast<const char*>(tstore) +
              (size_t)((col0 & 63) / BC) * (64 * BC) * sizeof(cplx<R>);
    v_ts = (uint32_t)((jt * BC + c0) * sizeof(cplx<R>));
    v_st = (uint32_t)(((size_t)jt * ncols + c0) * sizeof(cplx<R>));
  }
  // Row jt of tile row `trow` (a constant) whose store slot is s; every
  // choice below is wavefront-uniform.
  auto ts_load = [&](int trow, uint32_t s) {
    const bool h = ((tr.mask >> trow) & 1ull) != 0ull;
    const bool in = s < tcap;
    const char* sb =
        !h ? reinterpret_cast<const char*>(tw)
           : in ? ts_base + (size_t)s * (64 * 64 * sizeof(cplx<R>))
                : reinterpret_cast<const char*>(base) +
                      (size_t)trow * 64 * ncols * sizeof(cplx<R>);
    const cplx<R> v =
        *reinterpret_cast<const cplx<R>*>(sb + (size_t)(h && !in ? v_st : v_ts));
    return cplx<R>{h ? v.re : (R)0, h ? v.im : (R)0};
  };
  auto issue = [&](int n) {
    const int j = jt + (n / F0::RAD) * F0::TPC;
    if (F0::NB % F0::TPC == 0 || j < F0::NB) {
      const int e = j + (n % F0::RAD) * F0::NB;
      if constexpr (TS) {
        const int ta = ((n / F0::RAD) * F0::TPC + (n % F0::RAD) * F0::NB) / 64;
        qa[n] = ts_load(ta, __builtin_amdgcn_readlane(myslot, ta));
        qb[n] = ts_load(ta + NH / 64,
                        __builtin_amdgcn_readlane(myslot, ta + NH / 64));
      } else {
        qa[n] = tr.load(e, base + (size_t)e * ncols + c0, tw);
        qb[n] = tr.load(e + NH, base + (size_t)(e + NH) * ncols + c0, tw);
      }
    }
  };
#pragma unroll
  for (int n = 0; n < AHEAD && n < NE; ++n) issue(n);
  const auto twl = [&] {
    if constexpr (TABLE) {
      // The tables, while the first samples are in flight.
      for (int i = threadIdx.x; i < kTwLo + N / kTwLo; i += NT) {
        if (i < kTwLo) f_lo[i] = tw[i];
        else f_hi[i - kTwLo] = tw[(i - kTwLo) * kTwLo];
      }
      fill_stage_twiddles<R, LOGH, WIDE>(s_tab, tw, s, 2);
      __syncthreads();
      return TableTwiddles<R>{s_tab};
    } else {
      return Twiddles<R>{s_tab, s_tab + kTwLo};
    }
  }();
  const Twiddles<R> twf{f_lo, f_hi};
  auto ld_sum = [&](int e, int, int it, int r) {
    const int n = it * F0::RAD + r;
    if (n + AHEAD < NE) issue(n + AHEAD);
    const cplx<R> a = checker(qa[n], e);
    const cplx<R> b = checker(qb[n], e + NH);
    diff[it][r] = cmul(csub(a, b), twf(e, s));
    return cadd(a, b);
  };
  // Output 2e has the centring sign +1, output 2e + 1 the sign -1.
  auto st_even = [&](int e, int c, int, int, cplx<R> v) {
    base[(size_t)(2 * e) * ncols + c] = v;
  };
  fft_line<R, LOGH, BC, NT, WIDE>(lds, ld_sum, st_even, twl, s);
  auto ld_diff = [&](int, int, int it, int r) { return diff[it][r]; };
  auto st_odd = [&](int e, int c, int, int, cplx<R> v) {
    base[(size_t)(2 * e + 1) * ncols + c] = cplx<R>{-v.re, -v.im};
  };
  fft_line<R, LOGH, BC, NT, WIDE>(lds, ld_diff, st_odd, twl, s);
}

// ---- four-step column transform for long columns (N = N1 * N2) ---------
//
// Step A: for each n2, the length-N1 transform over rows n1*N2 + n2, times
// W_N^(n2 k1), written back to row k1*N2 + n2.  Step B: for each k1, the
// length-N2 transform over the contiguous rows k1*N2 + n2; output k2 is
// frequency q = k1 + N1 k2 and is written back in place to row k1*N2 + k2.
// Each step reads and writes the stack once with 16-column (128- or
// 256-byte) row segments; the result has its rows in the transposed order
// that stack_row() undoes.

// TM: rows of tiles without records (tile counts `tiles`, tile edge
// strip_w = 64) are not read: their loads go to `zeros`, a line of zeros
// (the one-call path leaves those tiles unwritten).  Choosing the address,
// not the loaded value, keeps the loads free of branches.
template <typename R, int LOG1, int LOG2, int BC, int NT, bool TM>
__global__ __launch_bounds__(NT) void k_fft_colA(
    cplx<R>* data, int ncols, int nplanes, const cplx<R>* __restrict__ tw, R s,
    const uint32_t* __restrict__ strips, int strip_w,
    const uint32_t* __restrict__ tiles, const cplx<R>* __restrict__ zeros) {
  constexpr int N1 = 1 << LOG1, N2 = 1 << LOG2, N = N1 * N2;
  __shared__ cplx<R> lds[lds_line<N1>(BC)];
  __shared__ cplx<R> s_lo[kTwLo], s_hi[(N1 + kTwLo - 1) / kTwLo];
  __shared__ uint32_t s_tm[TM ? N / 64 : 1];
  const int ncb = ncols / BC;
  const int nb = ncb * N2 * nplanes;
  const int L = xcd_block<R, BC>((int)blockIdx.x, nb);
  if (L >= nb) return;
  const int cb = L % ncb;
  const int rest = L / ncb;
  const int n2 = rest % N2;
  const int plane = rest / N2;
  if (strips != nullptr &&
      strips[plane * (ncols / strip_w) + cb * BC / strip_w] == 0u)
    return;
  cplx<R>* base = data + (size_t)plane * N * ncols + (size_t)cb * BC;
  if constexpr (TM) {
    // Record counts of the strip's tiles, one per 64 rows.
    const int tcols = ncols / 64, strip = cb * BC / 64;
    for (int i = (int)threadIdx.x; i < N / 64; i += NT)
      s_tm[i] = tiles[((size_t)plane * (N / 64) + i) * tcols + strip];
  }
  const Twiddles<R> twl = load_twiddles_sub(s_lo, s_hi, tw, N1, N);
  __syncthreads();
  auto ld = [&](int e, int c, int, int) {
    const int row = e * N2 + n2;
    if constexpr (TM) {
      const bool h = s_tm[row >> 6] != 0u;
      return checker(*(h ? base + (size_t)row * ncols + c : zeros), row);
    } else {
      return checker(base[(size_t)row * ncols + c], row);
    }
  };
  auto st = [&](int e, int c, int, int, cplx<R> v) {
    const int row = e * N2 + n2;
    base[(size_t)row * ncols + c] =
        cmul(v, twiddle_full(tw, (n2 * e) & (N - 1), s));
  };
  fft_line<R, LOG1, BC, NT>(lds, ld, st, twl, s);
}

template <typename R, int LOG1, int LOG2, int BC, int NT>
__global__ __launch_bounds__(NT) void k_fft_colB(
    cplx<R>* data, int ncols, int nplanes, const cplx<R>* __restrict__ tw, R s,
    const uint32_t* __restrict__ strips, int strip_w) {
  constexpr int N1 = 1 << LOG1, N2 = 1 << LOG2, N = N1 * N2;
  __shared__ cplx<R> lds[lds_line<N2>(BC)];
  __shared__ cplx<R> s_lo[kTwLo], s_hi[(N2 + kTwLo - 1) / kTwLo];
  const int ncb = ncols / BC;
  const int nb = ncb * N1 * nplanes;
  const int L = xcd_block<R, BC>((int)blockIdx.x, nb);
  if (L >= nb) return;
  const int cb = L % ncb;
  const int rest = L / ncb;
  const int k1 = rest % N1;
  const int plane = rest / N1;
  if (strips != nullptr &&
      strips[plane * (ncols / strip_w) + cb * BC / strip_w] == 0u)
    return;
  cplx<R>* base = data + (size_t)plane * N * ncols + (size_t)k1 * N2 * ncols +
                  (size_t)cb * BC;
  const Twiddles<R> twl = load_twiddles_sub(s_lo, s_hi, tw, N2, N);
  __syncthreads();
  auto ld = [&](int e, int c, int, int) { return base[(size_t)e * ncols + c]; };
  auto st = [&](int e, int c, int, int, cplx<R> v) {
    base[(size_t)e * ncols + c] = checker(v, k1 + N1 * e);
  };
  fft_line<R, LOG2, BC, NT>(lds, ld, st, twl, s);
}

// Undo the transposed row order of a four-step column transform: copy row
// r of the plane to row q(r) of the scratch plane.
template <typename R>
__global__ __launch_bounds__(256) void k_unpermute_rows(
    const cplx<R>* __restrict__ src, cplx<R>* __restrict__ dst, Geo g) {
  const int r = blockIdx.y;
  const int q = stack_freq(g, r);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < g.nu;
       i += gridDim.x * blockDim.x)
    dst[(size_t)q * g.nu + i] = src[(size_t)r * g.nu + i];
}

// ---- w-screen -------------------------------------------------------------

// exp(2 pi i a) for a phase a in turns, reduced to [-1/2, 1/2] in FP64.
__device__ __forceinline__ cplx<double> turns_phasor(double a) {
  const double f = a - rint(a);
  double sn, cs;
  sincospi(2.0 * f, &sn, &cs);
  return {cs, sn};
}

// n - 1 = sqrt(1 - l^2 - m^2) - 1 in the cancellation-free form.
__device__ __forceinline__ double n_minus_one(const Geo& g, int p, int q) {
  const double l = (double)(p - g.nu / 2) * g.dl;
  const double m = (double)(q - g.nv / 2) * g.dm;
  const double r2 = l * l + m * m;
  return -r2 / (1.0 + sqrt(1.0 - r2));
}

// Screen phasor exp(+-2 pi i w_k (n - 1)) of pixel (p, q), handed out plane
// by plane (k = 0, 1, ... in order, each once).  The phases w_0 (n - 1) and
// dw (n - 1) are formed and reduced to [-1/2, 1/2] turn in FP64 on both
// paths, and the phasor of plane 0 and the step between planes are taken
// from them with FP64 sincospi; each further plane's phasor is the
// previous one times the step (the planes are equispaced in w).  The FP64
// path advances an FP64 phasor; the FP32 path rounds the seed and step to
// FP32 and advances in FP32 (4 registers of state per pixel): its phase
// error grows by about one FP32 rounding per plane (~2e-6 rad after 32
// planes) and never sees the large unreduced argument.  `odd` adds half a
// turn to the seed: the output centring sign of odd pixels.
template <typename R>
struct Screen {
  cplx<R> ph, step;
  __device__ __forceinline__ void init(const Geo& g, int p, int q, bool conj,
                                       bool odd = false) {
    const double nm1 = n_minus_one(g, p, q);
    const cplx<double> a = turns_phasor(fma(g.w0, nm1, odd ? 0.5 : 0.0));
    const cplx<double> b = turns_phasor(g.dw * nm1);
    ph = {(R)a.re, (R)(conj ? -a.im : a.im)};
    step = {(R)b.re, (R)(conj ? -b.im : b.im)};
  }
  __device__ __forceinline__ cplx<R> next(const Geo&, int) {
    const cplx<R> w = ph;
    ph = cmul(ph, step);
    return w;
  }
};

// The step between planes of pixel (p, q), as Screen forms it, and the phase
// its rounding to FP32 adds per plane.
template <typename R>
__device__ __forceinline__ cplx<R> screen_step(const Geo& g, double nm1,
                                               R* drift) {
  const cplx<double> b = turns_phasor(g.dw * nm1);
  const cplx<R> s = {(R)b.re, (R)b.im};
  *drift = (R)((double)s.im * b.re - (double)s.re * b.im);
  return s;
}

// The phasor of plane 0; `odd` as for Screen.
__device__ __forceinline__ cplx<double> first_phase(const Geo& g, double nm1,
                                                    bool odd) {
  return turns_phasor(fma(g.w0, nm1, odd ? 0.5 : 0.0));
}

// The phasor ph of the first of `planes` planes, for steps rounded to FP32.
// Such a step is off by a factor 1 + e, plane k then by (1 + e)^k; the phasor
// takes (1 + e)^-c, c = (planes - 1) / 2, with it (to first order, e ~ 3e-8),
// so the error is that of half as many planes, either side of the middle one:
// a 4096^2 x 32 image 4.8e-7 -> 4.0e-7 off its 64-bit values.
template <typename R>
__device__ __forceinline__ cplx<R> centred(cplx<double> ph, int planes,
                                           cplx<R> step, R drift) {
  if constexpr (sizeof(R) == 4) {
    const double c = 0.5 * (double)(planes - 1);
    const double re = (double)step.re, im = (double)step.im;
    const double er = 1.0 - 0.5 * c * fma(re, re, fma(im, im, -1.0));
    const double ei = -c * (double)drift;
    ph = {ph.re * er - ph.im * ei, ph.re * ei + ph.im * er};
  }
  return {(R)ph.re, (R)ph.im};
}

// The plane sum sum_k F_k ph_0 step^k by Horner's rule, planes taken last
// to first: acc <- acc * step + F_k, and ph_0 * acc once at the end.  The
// same products as handing out ph_k (the contribution of plane k is
// multiplied by the step k times either way), in four fused multiply-adds
// per sample and plane instead of eight.
template <typename R>
__device__ __forceinline__ cplx<R> horner_step(cplx<R> acc, cplx<R> step,
                                               cplx<R> f) {
  return {fma(acc.re, step.re, fma(-acc.im, step.im, f.re)),
          fma(acc.re, step.im, fma(acc.im, step.re, f.im))};
}

// Grid correction of pixel (p, q): 1 / (c psi(f_p) psi(f_q)) from the
// plan's table, or 1 when the plan has none (uniform branch).  Imaging
// multiplies the plane sum by it; degridding multiplies its input image by
// it (the correction is real and diagonal, so it is its own adjoint).
template <typename R>
__device__ __forceinline__ cplx<R> corrected(const Geo& g, int p, int q,
                                             cplx<R> v) {
  if (g.corr == nullptr) return v;
  const R c = (R)(g.corr[p] * g.corr[g.nu + q]);
  return {v.re * c, v.im * c};
}

template <typename R>
__global__ __launch_bounds__(256) void k_wcorrect(const cplx<R>* __restrict__ F,
                                                  cplx<R>* __restrict__ img,
                                                  Geo g) {
  const int64_t pix = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npix = (int64_t)g.nu * g.nv;
  if (pix >= npix) return;
  const int q = (int)(pix / g.nu), p = (int)(pix - (int64_t)q * g.nu);
  Screen<R> sc;
  sc.init(g, p, q, false);
  cplx<R> acc = {(R)0, (R)0};
  const int64_t src = (int64_t)stack_row(g, q) * g.nu + p;
  for (int k = g.nw - 1; k >= 0; --k)
    acc = horner_step(acc, sc.step, F[(size_t)k * npix + src]);
  img[pix] = cadd(img[pix], corrected(g, p, q, cmul(sc.ph, acc)));
}

// Shape of the fused row kernels.
//   NT     threads a line: 8 points each, and radix-8 stages, so that 16
//          wavefronts (FP32) share a CU.  4096 x 4096 x 32 planes, ms: FP32
//          0.96 (16 points each and radix-16 stages: fewer LDS exchanges but
//          half the wavefronts, 1.01), FP64 1.96.  8192-point FP32 lines take
//          16 points and radix 16 (one workgroup of 512 threads either way,
//          one stage less).
//   GMAX   lines (planes of one row) a workgroup, where the image has too few
//          rows to fill the device
//   TABLE  stage twiddles held whole (RowTwiddles); beyond 4096 points lookup
//          tables
//   FITS   the kernels exist: a line and the tables in one workgroup's LDS,
//          and 16 wavefronts of registers
//   SUMS   the summing kernel too: its accumulators and steps spill at 1024
//          threads (8192-point FP64 rows of 8 planes 6.6 ms; unfused 5.3)
constexpr int row_nt(int real_bytes, int logn) {
  const int per = real_bytes == 4 && logn == 13 ? 4 : 3;
  return logn - per < 6 ? 64 : 1 << (logn - per);
}
// Wavefronts per SIMD the register budget has to allow (two FP32 workgroups
// of 512 threads a CU).
constexpr int row_waves(int real_bytes, int logn) {
  return real_bytes == 4 && logn >= 9 && logn <= 12 ? 4 : 1;
}
template <typename R, int LOGN>
struct RowShape {
  static constexpr bool WIDE = sizeof(R) == 4 && LOGN == 13;
  static constexpr int N = 1 << LOGN;
  static constexpr int NT = row_nt(sizeof(R), LOGN);
  static constexpr int GMAX = NT >= 256 ? 1 : 512 / NT;
  static constexpr bool TABLE = LOGN <= 12;
  static constexpr int TAB =
      TABLE ? (RowTwiddles<R, LOGN, NT>::kTab > 0
                   ? RowTwiddles<R, LOGN, NT>::kTab : 1)
            : kTwLo + (N + kTwLo - 1) / kTwLo;
  static constexpr bool FITS = LOGN <= 13;
  static constexpr bool SUMS = FITS && NT <= 512;
};

// Twiddles of a fused row kernel, with s_tab (RowShape::TAB entries) in LDS.
// RowTwiddles hold the input centring; lookup tables leave it to the caller
// (odd elements negated as they are loaded).
template <typename R, int LOGN>
__device__ __forceinline__ auto row_twiddles(cplx<R>* s_tab,
                                             const cplx<R>* tw, R s,
                                             int tid) {
  using RS = RowShape<R, LOGN>;
  if constexpr (RS::TABLE) {
    static_assert(!RS::WIDE, "RowTwiddles are radix 8");
    return RowTwiddles<R, LOGN, RS::NT>(s_tab, tw, s, tid);
  } else {
    return load_twiddles(s_tab, s_tab + kTwLo, tw, RS::N);
  }
}

// Row transform of every plane + screen + plane sum into image row q.
//
// A workgroup transforms G planes of its row at a time (group gi of NT
// threads takes planes [gi * per, ...), last to first: Horner's rule,
// horner_step) and sums the groups' parts in order at the end; G > 1 is for
// images of few rows, whose serial chain of planes would otherwise leave the
// device idle.
//
// Bound by LDS and vector issue together: a 4096-point FP32 line and plane
// takes 4500 cycles of a CU, in which the LDS is active for 2040 (512 of them
// bank conflicts) and 3500 vector instructions issue, 0.7 cycles each.  The
// row of the next plane is in flight while one is transformed, the strip
// marks are bits of a wavefront mask read one plane earlier, and the largest
// stage's twiddles are not read again for each plane (RowTwiddles).  4096 x
// 4096 x 32 planes: FP32 1.07 -> 0.95 ms, FP64 2.42 -> 1.95.
// 8192 points fused: 32 planes of 8192^2 FP32 10.3 (rows, then screen) -> 5.2.
template <typename R, int LOGN, int G>
__global__ __launch_bounds__(row_nt(sizeof(R), LOGN) * G, row_waves(sizeof(R), LOGN))
    void k_row_screen_sum(const cplx<R>* __restrict__ planes,
                          cplx<R>* __restrict__ img, Geo g,
                          const cplx<R>* __restrict__ tw,
                          const uint32_t* __restrict__ strips) {
  using RS = RowShape<R, LOGN>;
  constexpr int N = RS::N, NT = RS::NT;
  constexpr bool WIDE = RS::WIDE;
  using L = Stage<R, LOGN, 1, NT, stage_npass(LOGN, WIDE) - 1, WIDE>;
  constexpr int IT = L::IT, RAD = L::RAD, NB = L::NB;
  __shared__ cplx<R> lds_all[G][lds_line<N>(1)];
  __shared__ __align__(16) cplx<R> s_tab[RS::TAB];
  __shared__ cplx<R> s_step[G > 1 ? N : 1];
  // FP32: the phasors of plane 0, where that leaves as many workgroups per CU
  // as the registers do (16 wavefronts; not 1024 points with G = 1: seven of
  // eight).
  constexpr bool SEEDS =
      sizeof(R) == 4 &&
      (LOGN == 13 || (sizeof(lds_all) + sizeof(s_tab) + sizeof(s_step) +
                      N * sizeof(cplx<R>)) * (1024 / (NT * G)) <= 160 * 1024);
  __shared__ cplx<R> s_seed[SEEDS ? N : 1];
  const int q = blockIdx.x;
  const int gi = G == 1 ? 0 : (int)uniform_u32(threadIdx.x / NT);
  const int tid = G == 1 ? (int)threadIdx.x : (int)threadIdx.x % NT;
  cplx<R>* lds = lds_all[gi];
  const auto twl = row_twiddles<R, LOGN>(s_tab, tw, (R)1, tid);
  __syncthreads();
  // The output centring (-1)^p is half a turn in the screen phase.
  const int per = (g.nw + G - 1) / G;
  const int k0 = gi * per, k1 = min(k0 + per, g.nw);
  cplx<R> acc[IT][RAD], step[IT][RAD];
  // Steps (and FP32 seeds) of the row's pixels, once per workgroup and in a
  // rolled loop: unrolled over a thread's pixels the FP64 functions spill.
  cplx<R>* steps = G > 1 ? s_step : lds;
  if constexpr (G > 1 || SEEDS) {
    for (int p = threadIdx.x; p < N; p += NT * G) {
      const double nm1 = n_minus_one(g, p, q);
      R drift;
      steps[p] = screen_step<R>(g, nm1, &drift);
      if constexpr (SEEDS)
        s_seed[p] = centred<R>(first_phase(g, nm1, (p & 1) != 0), g.nw,
                               steps[p], drift);
    }
    __syncthreads();
  }
#pragma unroll
  for (int it = 0; it < IT; ++it)
#pragma unroll
    for (int r = 0; r < RAD; ++r) {
      const int j = tid + it * NT, p = j + r * NB;
      acc[it][r] = {(R)0, (R)0};
      step[it][r] = {(R)1, (R)0};
      if (NB % NT == 0 || j < NB) {
        if constexpr (G > 1 || SEEDS) {
          step[it][r] = steps[p];
        } else {
          R drift;
          step[it][r] = screen_step<R>(g, n_minus_one(g, p, q), &drift);
        }
      }
    }
  if constexpr (G == 1 && SEEDS) __syncthreads();  // lds is the line again
  auto seed = [&](int p) -> cplx<R> {
    if constexpr (SEEDS) return s_seed[p];
    const cplx<double> a = first_phase(g, n_minus_one(g, p, q), (p & 1) != 0);
    return {(R)a.re, (R)a.im};
  };
  using F0 = Stage<R, LOGN, 1, NT, 0, WIDE>;
  constexpr int IT0 = F0::IT, RAD0 = F0::RAD, NB0 = F0::NB;
  // Column-strip marks (64-column strips, T = 64) as bits: samples of strips
  // that hold no data are not read and taken as zero.  The row of the next
  // plane is requested as the first stage takes the current one from
  // registers, the marks of the plane after that one plane earlier still.
  constexpr int MW = (N + 4095) / 4096;
  constexpr bool kUniform = NB0 % 64 == 0 && NT % 64 == 0;
  const bool skip = g.T == 64;
  const int lane = (int)threadIdx.x & 63;
  const size_t row = (size_t)stack_row(g, q) * N;
  uint32_t mk[MW];
  unsigned long long mask[MW];
  auto load_marks = [&](int n) {
    const int k = k0 + n;
    const bool in = n >= 0 && k < k1;
#pragma unroll
    for (int w = 0; w < MW; ++w) {
      mk[w] = in ? 1u : 0u;
      if (skip && in)
        mk[w] = strips[(size_t)k * g.tiles_u +
                       min(w * 64 + lane, g.tiles_u - 1)];
    }
  };
  auto take_marks = [&]() {
#pragma unroll
    for (int w = 0; w < MW; ++w) mask[w] = __ballot(mk[w] != 0u);
  };
  cplx<R> buf[IT0][RAD0];
  auto request = [&](int n, int it, int r) {
    const int j = tid + it * NT;
    buf[it][r] = {(R)0, (R)0};
    if (NB0 % NT == 0 || j < NB0) {
      const int e = j + r * NB0;
      const int sb = kUniform ? (int)uniform_u32(e >> 6) : e >> 6;
      if ((mask[MW > 1 ? sb >> 6 : 0] >> (sb & 63)) & 1ull) {
        const cplx<R>* line = planes + (size_t)(k0 + n) * g.nv * N + row;
        // FP32 rows of RowTwiddles: a scalar base and the thread's index, or
        // the addresses of the thread's samples take registers that the
        // factors need (8192 points, without them: 5.21 -> 5.37 ms).
        if constexpr (sizeof(R) == 4 && RS::TABLE)
          buf[it][r] = uniform_ptr(line + it * NT + r * NB0)[(uint32_t)tid];
        else
          buf[it][r] = line[e];
      }
    }
  };
  load_marks(per - 1);
  take_marks();
#pragma unroll
  for (int it = 0; it < IT0; ++it)
#pragma unroll
    for (int r = 0; r < RAD0; ++r) request(per - 1, it, r);
  load_marks(per - 2);
  for (int n = per - 1; n >= 0; --n) {
    take_marks();  // of plane n - 1
    load_marks(n - 2);
    auto ld = [&](int e, int, int it, int r) {
      const cplx<R> v = buf[it][r];
      request(n - 1, it, r);
      return RS::TABLE ? v : checker(v, e);
    };
    auto st = [&](int, int, int it, int r, cplx<R> v) {
      acc[it][r] = horner_step(acc[it][r], step[it][r], v);
    };
    fft_line<R, LOGN, 1, NT, WIDE>(lds, ld, st, twl, (R)1, tid);
  }
  cplx<R>* out = img + (size_t)q * N;
  if constexpr (G == 1) {
    // Add into the image row: all reads first, then all writes.
    cplx<R> old[IT][RAD];
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int r = 0; r < RAD; ++r) {
        const int j = tid + it * NT;
        if (NB % NT == 0 || j < NB) old[it][r] = out[j + r * NB];
      }
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int r = 0; r < RAD; ++r) {
        const int j = tid + it * NT, p = j + r * NB;
        if (NB % NT == 0 || j < NB)
          out[p] = cadd(old[it][r],
                        corrected(g, p, q,
                                  cmul(seed(p), acc[it][r])));
      }
  } else {
    // Group u's part belongs at step^(u per): Horner's rule once more, over
    // the groups.
    __syncthreads();  // the last stage's reads are done
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
      for (int r = 0; r < RAD; ++r) {
        const int j = tid + it * NT;
        if (NB % NT == 0 || j < NB) lds[j + r * NB] = acc[it][r];
      }
    __syncthreads();
    for (int p = threadIdx.x; p < N; p += NT * G) {
      const cplx<R> s1 = s_step[p];
      cplx<R> sp = s1;
      for (int i = 1; i < per; ++i) sp = cmul(sp, s1);
      cplx<R> sum = lds_all[G - 1][p];
#pragma unroll
      for (int u = G - 2; u >= 0; --u)
        sum = horner_step(sum, sp, lds_all[u][p]);
      out[p] = cadd(out[p],
                    corrected(g, p, q,
                              cmul(seed(p), sum)));
    }
  }
}

// Degridding counterpart: image row q times each plane's conjugate screen,
// then the row transform (sign -1), written to row q of every plane.  The
// planes are cut into gridDim.y runs, for images of few rows.
template <typename R, int LOGN>
__global__ __launch_bounds__(row_nt(sizeof(R), LOGN), row_waves(sizeof(R), LOGN))
    void k_screen_row_bcast(const void* __restrict__ img, int img_real,
                            cplx<R>* __restrict__ planes, Geo g,
                            const cplx<R>* __restrict__ tw) {
  using RS = RowShape<R, LOGN>;
  constexpr int N = RS::N, NT = RS::NT;
  constexpr bool WIDE = RS::WIDE;
  using F0 = Stage<R, LOGN, 1, NT, 0, WIDE>;
  constexpr int IT = F0::IT, RAD = F0::RAD, NB = F0::NB;
  __shared__ cplx<R> lds[lds_line<N>(1)];
  __shared__ __align__(16) cplx<R> s_tab[RS::TAB];
  const int q = blockIdx.x;
  const auto twl = row_twiddles<R, LOGN>(s_tab, tw, (R)-1,
                                          (int)threadIdx.x);
  __syncthreads();
  const int per = (g.nw + gridDim.y - 1) / gridDim.y;
  const int k0 = (int)blockIdx.y * per, k1 = min(k0 + per, g.nw);
  // x: the pixel times the conjugate screen of the next plane.
  cplx<R> x[IT][RAD], step[IT][RAD];
#pragma unroll
  for (int it = 0; it < IT; ++it)
#pragma unroll
    for (int r = 0; r < RAD; ++r) {
      const int j = threadIdx.x + it * NT;
      x[it][r] = {(R)0, (R)0};
      step[it][r] = {(R)1, (R)0};
      if (NB % NT == 0 || j < NB) {
        const int p = j + r * NB;
        cplx<R> v = {(R)0, (R)0};
        if (img_real) {
          v.re = reinterpret_cast<const R*>(img)[(size_t)q * N + p];
        } else {
          v = reinterpret_cast<const cplx<R>*>(img)[(size_t)q * N + p];
        }
        // The phasor of plane k0, its phase formed in FP64.
        const double nm1 = n_minus_one(g, p, q);
        const cplx<double> ph =
            turns_phasor(fma((double)k0, g.dw, g.w0) * nm1);
        R drift;
        const cplx<R> b = screen_step<R>(g, nm1, &drift);
        const cplx<R> a = centred<R>(ph, k1 - k0, b, drift);
        x[it][r] = cmul(corrected(g, p, q, v), cplx<R>{a.re, -a.im});
        step[it][r] = {b.re, -b.im};
      }
    }
  for (int k = k0; k < k1; ++k) {
    cplx<R>* line = planes + ((size_t)k * g.nv + q) * N;
    auto ld = [&](int e, int, int it, int r) {
      const cplx<R> v = x[it][r];
      x[it][r] = cmul(v, step[it][r]);
      return RS::TABLE ? v : checker(v, e);
    };
    // The output centring stays on the stores (the column transform that
    // follows centres the other axis).
    auto st = [&](int e, int, int, int, cplx<R> v) { line[e] = checker(v, e); };
    fft_line<R, LOGN, 1, NT, WIDE>(lds, ld, st, twl, (R)-1);
  }
}

// Degridding, any grid size: plane k = image * conj(screen_k), natural
// row order, one pixel per thread across all planes.
template <typename R>
__global__ __launch_bounds__(256) void k_screen_bcast(
    const void* __restrict__ img, int img_real, cplx<R>* __restrict__ planes,
    Geo g) {
  const int64_t pix = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t npix = (int64_t)g.nu * g.nv;
  if (pix >= npix) return;
  const int q = (int)(pix / g.nu), p = (int)(pix - (int64_t)q * g.nu);
  cplx<R> x = {(R)0, (R)0};
  if (img_real) x.re = reinterpret_cast<const R*>(img)[pix];
  else x = reinterpret_cast<const cplx<R>*>(img)[pix];
  x = corrected(g, p, q, x);
  Screen<R> sc;
  sc.init(g, p, q, true);
  for (int k = 0; k < g.nw; ++k) {
    const auto w = sc.next(g, k);
    planes[(size_t)k * npix + pix] = cmul(x, cplx<R>{(R)w.re, (R)w.im});
  }
}

template <typename R>
__global__ __launch_bounds__(256) void k_fill_zero(cplx<R>* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = i; t < n; t += stride) p[t] = cplx<R>{(R)0, (R)0};
}

__global__ __launch_bounds__(256) void k_fill_zero_u32(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = i; t < n; t += stride) p[t] = 0u;
}

// A plan's tables, one thread per entry of an axis (u, then v): the
// twiddles e^{2 pi i idx / n}; with g.corr, the grid-correction factors 1 /
// (c psi(f)) along u and 1 / psi(f) along v; and the 256 bytes of zeros.
// One launch: the allocation-free call fills them anew each time.
template <typename R>
__global__ __launch_bounds__(64) void k_tables(Geo g, cplx<R>* tw_u,
                                               cplx<R>* tw_v, double* corr,
                                               uint32_t* zeros) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 64) zeros[i] = 0u;
  if (i >= g.nu + g.nv) return;
  const bool u = i < g.nu;
  const int n = u ? g.nu : g.nv;
  const int idx = u ? i : i - g.nu;
  double sn, cs;
  sincospi(2.0 * (double)idx / (double)n, &sn, &cs);
  (u ? tw_u : tw_v)[idx] = cplx<R>{(R)cs, (R)sn};
  if (g.corr == nullptr) return;
  const double f = (double)(idx - n / 2) / (double)n;
  const double psi = kernel_transform(g.kern, g.K, g.inv2s2, g.es_beta, f);
  corr[i] = 1.0 / ((u ? g.cnorm : 1.0) * psi);
}

// Threads per row transform: enough to cover the N/8 first-stage
// butterflies once, 64..512.
constexpr int row_threads(int logn) {
  return (1 << logn) / 8 < 64 ? 64 : ((1 << logn) / 8 > 512 ? 512 : (1 << logn) / 8);
}

// A whole line of 2^LOGN elements of type R fits one workgroup's LDS.
template <typename R, int LOGN>
constexpr bool line_fits() {
  return lds_line<(1 << LOGN)>(1) * (int)sizeof(cplx<R>) <= 150 * 1024;
}

template <typename R, int LOGN>
bool rows_t(cplx<R>* data, int64_t nrows, const cplx<R>* tw, R s,
            cplx<R>* scratch, const uint32_t* strips, int rows_per_plane,
            int strips_per_row, hipStream_t st) {
  if constexpr (line_fits<R, LOGN>()) {
    constexpr int NT = row_threads(LOGN);
    if (strips == nullptr) {
      hipLaunchKernelGGL((k_fft_rows<R, LOGN, NT, false>),
                         dim3((unsigned)nrows), dim3(NT), 0, st, data, nrows,
                         tw, s, strips, rows_per_plane, strips_per_row);
      return true;
    }
    // Shorter rows are fused with the screen (RowShape).
    if constexpr (!RowShape<R, LOGN>::SUMS && NT % 64 == 0 &&
                  ((1 << LOGN) / 8) % 64 == 0) {
      hipLaunchKernelGGL((k_fft_rows<R, LOGN, NT, true>),
                         dim3((unsigned)nrows), dim3(NT), 0, st, data, nrows,
                         tw, s, strips, rows_per_plane, strips_per_row);
      return true;
    }
    return false;
  } else if constexpr (line_fits<R, LOGN - 1>()) {
    constexpr int NT = row_threads(LOGN - 1);
    if (strips == nullptr) {
      hipLaunchKernelGGL((k_fft_rows_split<R, LOGN - 1, NT, false>),
                         dim3((unsigned)nrows), dim3(NT), 0, st, data, nrows,
                         tw, s, strips, rows_per_plane, strips_per_row);
      return true;
    }
    if constexpr (NT % 64 == 0 && ((1 << (LOGN - 1)) / 8) % 64 == 0) {
      hipLaunchKernelGGL((k_fft_rows_split<R, LOGN - 1, NT, true>),
                         dim3((unsigned)nrows), dim3(NT), 0, st, data, nrows,
                         tw, s, strips, rows_per_plane, strips_per_row);
      return true;
    }
    return false;
  } else if constexpr (line_fits<R, LOGN - 2>()) {
    if (scratch == nullptr || strips != nullptr) return false;
    constexpr int NT = row_threads(LOGN - 2);
    const int64_t g = nrows < kSplitRowGroups ? nrows : kSplitRowGroups;
    hipLaunchKernelGGL((k_fft_rows_splitF<R, LOGN - 2, NT, 4>),
                       dim3((unsigned)(g > 0 ? g : 1)), dim3(NT), 0, st, data,
                       nrows, tw, s, scratch);
    return true;
  } else {
    return false;
  }
}

int ilog2(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

template <typename R, int LOGN>
bool cols_t(cplx<R>* data, int ncols, int nplanes, const cplx<R>* tw, R s,
            const uint32_t* strips, int strip_w, const uint32_t* tiles,
            const cplx<R>* tstore, const uint32_t* tslot, uint32_t tcap,
            hipStream_t st) {
  if constexpr (LOGN > 12) {
    return false;
  } else {
  constexpr int N = 1 << LOGN;
  constexpr int ELEM = sizeof(cplx<R>);
  // Strips and tile rows are powers of two; a tile table covers at most
  // 64 tile rows (one bit each in a wavefront mask).
  const bool pow2 = strip_w > 0 && (strip_w & (strip_w - 1)) == 0;
  if (!pow2) {
    if (tiles != nullptr) return false;
    strips = nullptr;
  }
  const int log_strip = pow2 ? ilog2(strip_w) : 0;
  if (tiles != nullptr && (N >> log_strip) > 64) return false;
  // Widest column block (<= 16) whose padded N x BC tile fits 150 KiB of
  // LDS (the twiddle tables take the rest).
  constexpr int BCMAX = (150 * 1024) / (lds_line<N>(1) * ELEM);
  constexpr int BC = BCMAX >= 16 ? 16 : (BCMAX >= 8 ? 8 : (BCMAX >= 4 ? 4 : (BCMAX >= 2 ? 2 : 1)));
  constexpr int NT = (N * BC) / 8 < 64 ? 64 : ((N * BC) / 8 > 1024 ? 1024 : (N * BC) / 8);
  const int nb = (ncols / BC) * nplanes;
  const int grid = ((nb + 7) / 8) * 8;
  if constexpr (BC * ELEM < 128 && LOGN >= 10) {
    // Twice the columns per block with the split transform.
    constexpr int BC2 = 2 * BC;
    // FP32: 512 threads (256 registers each: a deeper queue of loads per
    // wavefront beats more wavefronts; measured 25% faster than 1024 at
    // 4096-point columns); FP64: 1024.
    constexpr int CAP = sizeof(R) == 4 ? 512 : 1024;
    constexpr int NT2 = (N / 2 * BC2) / 8 > CAP ? CAP : (N / 2 * BC2) / 8;
    if (ncols % BC2 == 0) {
      const int nb2 = (ncols / BC2) * nplanes;
      if (strip_w % BC2 != 0) {
        if (tiles != nullptr) return false;  // the table cannot be honoured
        strips = nullptr;
      }
      if constexpr (BC2 * ELEM == 64 && NT2 / BC2 == 64 && LOGN >= 7) {
        if (tstore != nullptr) {
          if (tiles == nullptr || strips == nullptr || strip_w != 64)
            return false;
          hipLaunchKernelGGL((k_fft_cols_split<R, LOGN - 1, BC2, NT2, true>),
                             dim3(((nb2 + 7) / 8) * 8), dim3(NT2), 0, st,
                             data, ncols, nplanes, tw, s, strips, log_strip,
                             tiles, tstore, tslot, tcap);
          return true;
        }
      }
      if (tstore != nullptr) return false;
      hipLaunchKernelGGL((k_fft_cols_split<R, LOGN - 1, BC2, NT2, false>),
                         dim3(((nb2 + 7) / 8) * 8), dim3(NT2), 0, st, data,
                         ncols, nplanes, tw, s, strips, log_strip, tiles,
                         (const cplx<R>*)nullptr, (const uint32_t*)nullptr,
                         0u);
      return true;
    }
  }
  if (tstore != nullptr) return false;
  if (strip_w % BC != 0) {
    if (tiles != nullptr) return false;
    strips = nullptr;
  }
  hipLaunchKernelGGL((k_fft_cols<R, LOGN, BC, NT>), dim3(grid), dim3(NT), 0,
                     st, data, ncols, nplanes, tw, s, strips, log_strip, tiles);
  return true;
  }
}

template <typename R, int LOG1, int LOG2, int BC>
bool cols4_bc(cplx<R>* data, int ncols, int nplanes, const cplx<R>* tw, R s,
              const uint32_t* strips, int strip_w, const uint32_t* tiles,
              const cplx<R>* zeros, hipStream_t st) {
  constexpr int NTA = ((1 << LOG1) * BC) / 8;
  constexpr int NTB = ((1 << LOG2) * BC) / 8;
  static_assert(NTA <= 1024 && NTB <= 1024, "step too long for one block");
  const int ncb = ncols / BC;
  const int nba = ncb * (1 << LOG2) * nplanes;
  const int nbb = ncb * (1 << LOG1) * nplanes;
  if (strips != nullptr && strip_w % BC != 0) strips = nullptr;
  if (tiles != nullptr) {
    // Tile counts need strips of 64 columns holding whole blocks.
    if (strips == nullptr || strip_w != 64 || 64 % BC != 0 ||
        zeros == nullptr)
      return false;
    hipLaunchKernelGGL((k_fft_colA<R, LOG1, LOG2, BC, NTA, true>),
                       dim3(((nba + 7) / 8) * 8), dim3(NTA), 0, st, data,
                       ncols, nplanes, tw, s, strips, strip_w, tiles, zeros);
  } else {
    hipLaunchKernelGGL((k_fft_colA<R, LOG1, LOG2, BC, NTA, false>),
                       dim3(((nba + 7) / 8) * 8), dim3(NTA), 0, st, data,
                       ncols, nplanes, tw, s, strips, strip_w, tiles, zeros);
  }
  hipLaunchKernelGGL((k_fft_colB<R, LOG1, LOG2, BC, NTB>),
                     dim3(((nbb + 7) / 8) * 8), dim3(NTB), 0, st, data, ncols,
                     nplanes, tw, s, strips, strip_w);
  return true;
}

template <typename R, int LOGN>
bool cols4_t(cplx<R>* data, int ncols, int nplanes, const cplx<R>* tw, R s,
             const uint32_t* strips, int strip_w, const uint32_t* tiles,
             const cplx<R>* zeros, hipStream_t st) {
  if constexpr (LOGN < 6) {
    return false;
  } else {
    constexpr int LOG1 = LOGN / 2, LOG2 = LOGN - LOG1;
    // 512-byte row segments (64 FP32 or 32 FP64 columns) per workgroup
    // when the grid is that wide (fewer if a step would exceed 1024
    // threads); 16 columns otherwise.
    constexpr int BCW = 512 / (int)sizeof(cplx<R>);
    constexpr int NMAX = (1 << LOG2) > (1 << LOG1) ? (1 << LOG2) : (1 << LOG1);
    constexpr int BC = (NMAX * BCW) / 8 > 1024 ? (8 * 1024) / NMAX : BCW;
    if (ncols >= BC && ncols % BC == 0)
      return cols4_bc<R, LOG1, LOG2, BC>(data, ncols, nplanes, tw, s, strips,
                                         strip_w, tiles, zeros, st);
    return cols4_bc<R, LOG1, LOG2, 16>(data, ncols, nplanes, tw, s, strips,
                                       strip_w, tiles, zeros, st);
  }
}

// Wavefronts a launch should have at least: what FP32 kernels of 128 registers
// fill the device's 1024 SIMDs with.  Row sums at 1024 / 2048 / 4096 / 8192, us:
// 1024^2 x 16 FP32 50 / 50 / 41 / 43, 512^2 x 8 FP64 18.0 / 16.7 / 18.7 / 18.7,
// 128^2 x 4 and 2048^2 x 16 the same; broadcast of 256^2 x 8 FP64 17.7 / 19.7 /
// 19.5 / 20.0.
constexpr int64_t kEnoughWaves = 4096;

template <typename R, int LOGN, int G>
void row_screen_g(const cplx<R>* planes, cplx<R>* img, const Geo& g,
                  const cplx<R>* tw, const uint32_t* strips, hipStream_t st) {
  hipLaunchKernelGGL((k_row_screen_sum<R, LOGN, G>), dim3(g.nv),
                     dim3(RowShape<R, LOGN>::NT * G), 0, st, planes, img, g,
                     tw, strips);
}

template <typename R, int LOGN>
bool row_screen_t(const cplx<R>* planes, cplx<R>* img, const Geo& g,
                  const cplx<R>* tw, const uint32_t* strips, hipStream_t st) {
  using RS = RowShape<R, LOGN>;
  if constexpr (!RS::SUMS) {
    return false;
  } else {
    constexpr int GM = RS::GMAX;
    const int64_t waves = (int64_t)g.nv * RS::NT / 64;
    // Half the groups where that fills the device, or the planes run out.
    if constexpr (GM >= 4) {
      if (g.nw > 2 && waves * 2 < kEnoughWaves) {
        if (GM > 4 && (g.nw <= 4 || waves * 4 >= kEnoughWaves))
          row_screen_g<R, LOGN, 4>(planes, img, g, tw, strips, st);
        else
          row_screen_g<R, LOGN, GM>(planes, img, g, tw, strips, st);
        return true;
      }
    }
    if constexpr (GM >= 2) {
      if (g.nw > 1 && waves < kEnoughWaves) {
        row_screen_g<R, LOGN, 2>(planes, img, g, tw, strips, st);
        return true;
      }
    }
    row_screen_g<R, LOGN, 1>(planes, img, g, tw, strips, st);
    return true;
  }
}

template <typename R, int LOGN>
bool screen_bcast_t(const void* img, int img_real, cplx<R>* planes,
                    const Geo& g, const cplx<R>* tw, hipStream_t st) {
  using RS = RowShape<R, LOGN>;
  if constexpr (!RS::FITS) {
    return false;
  } else {
    int runs = 1;
    while (runs * 2 <= g.nw &&
           (int64_t)g.nv * RS::NT / 64 * runs < kEnoughWaves)
      runs *= 2;
    hipLaunchKernelGGL((k_screen_row_bcast<R, LOGN>), dim3(g.nv, runs),
                       dim3(RS::NT), 0, st, img, img_real, planes, g, tw);
    return true;
  }
}

#define WS_LOGN_SWITCH(LOGN_VAR, CALL)                                     \
  switch (LOGN_VAR) {                                                      \
    case 4: { constexpr int LG = 4; CALL; } break;                         \
    case 5: { constexpr int LG = 5; CALL; } break;                         \
    case 6: { constexpr int LG = 6; CALL; } break;                         \
    case 7: { constexpr int LG = 7; CALL; } break;                         \
    case 8: { constexpr int LG = 8; CALL; } break;                         \
    case 9: { constexpr int LG = 9; CALL; } break;                         \
    case 10: { constexpr int LG = 10; CALL; } break;                       \
    case 11: { constexpr int LG = 11; CALL; } break;                       \
    case 12: { constexpr int LG = 12; CALL; } break;                       \
    case 13: { constexpr int LG = 13; CALL; } break;                       \
    case 14: { constexpr int LG = 14; CALL; } break;                       \
    case 15: { constexpr int LG = 15; CALL; } break;                       \
    default: return false;                                                 \
  }

}  // namespace

bool fft_supported(int n, int elem_bytes) {
  // A quarter row must fit one workgroup's LDS (150 KiB with padding).
  return n >= 16 && n <= 32768 && (n & (n - 1)) == 0 &&
         (size_t)(n / 4 + n / 128) * elem_bytes <= 150 * 1024;
}

bool fft_row_needs_scratch(int n, int elem_bytes) {
  // Rows longer than two half-length LDS transforms take the 4-way split.
  return (size_t)(n / 2 + n / 64) * elem_bytes > 150 * 1024;
}

size_t fft_row_scratch_bytes(int n, int elem_bytes) {
  return fft_row_needs_scratch(n, elem_bytes)
             ? (size_t)kSplitRowGroups * n * elem_bytes : 0;
}

// The plain row transforms read by strip marks when one wavefront's 64
// first-stage samples lie in one strip: the one-pass and two-half forms of
// rows too long to be fused, not the 4-way split.
bool fft_rows_can_mask(int n, int elem_bytes) {
  return fft_supported(n, elem_bytes) && !rows_can_fuse(n, elem_bytes) &&
         !fft_row_needs_scratch(n, elem_bytes);
}

bool rows_can_fuse(int n, int elem_bytes) {
  return n <= (elem_bytes == 16 ? 4096 : 8192);
}

bool rows_can_bcast(int n, int) { return n <= 8192; }

template <typename R>
bool launch_fft_rows(void* data, int n, int64_t nrows, const void* tw, int sign,
                     void* scratch, const uint32_t* strips, int rows_per_plane,
                     hipStream_t st) {
  const int lg = ilog2(n);
  bool ok = false;
  WS_LOGN_SWITCH(lg, (ok = rows_t<R, LG>((cplx<R>*)data, nrows,
                                         (const cplx<R>*)tw, (R)sign,
                                         (cplx<R>*)scratch, strips,
                                         rows_per_plane, n / 64, st)));
  return ok;
}

template <typename R>
bool launch_fft_cols(void* data, int nrows, int ncols, int nplanes,
                     const void* tw, int sign, const uint32_t* strips,
                     int strip_w, const uint32_t* tiles, const void* tstore,
                     const uint32_t* tslot, uint32_t tcap, hipStream_t st) {
  const int lg = ilog2(nrows);
  bool ok = false;
  WS_LOGN_SWITCH(lg, (ok = cols_t<R, LG>((cplx<R>*)data, ncols, nplanes,
                                         (const cplx<R>*)tw, (R)sign, strips,
                                         strip_w, tiles,
                                         (const cplx<R>*)tstore, tslot, tcap,
                                         st)));
  return ok;
}

template <typename R>
bool launch_row_screen_sum(const void* planes, void* img, const Geo& g,
                           const void* tw_u, const uint32_t* strips,
                           hipStream_t st) {
  const int lg = ilog2(g.nu);
  bool ok = false;
  WS_LOGN_SWITCH(lg, (ok = row_screen_t<R, LG>((const cplx<R>*)planes,
                                               (cplx<R>*)img, g,
                                               (const cplx<R>*)tw_u, strips,
                                               st)));
  return ok;
}

template <typename R>
bool launch_screen_row_bcast(const void* img, int img_real, void* planes,
                             const Geo& g, const void* tw_u, hipStream_t st) {
  const int lg = ilog2(g.nu);
  bool ok = false;
  WS_LOGN_SWITCH(lg, (ok = screen_bcast_t<R, LG>(img, img_real,
                                                 (cplx<R>*)planes, g,
                                                 (const cplx<R>*)tw_u, st)));
  return ok;
}

template <typename R>
bool launch_fft_cols4(void* data, int nrows, int ncols, int nplanes,
                      const void* tw, int sign, const uint32_t* strips,
                      int strip_w, const uint32_t* tiles, const void* zeros,
                      hipStream_t st) {
  const int lg = ilog2(nrows);
  bool ok = false;
  WS_LOGN_SWITCH(lg, (ok = cols4_t<R, LG>((cplx<R>*)data, ncols, nplanes,
                                          (const cplx<R>*)tw, (R)sign, strips,
                                          strip_w, tiles,
                                          (const cplx<R>*)zeros, st)));
  return ok;
}

template <typename R>
void launch_unpermute_rows(const void* src, void* dst, const Geo& g,
                           hipStream_t st) {
  const int bx = (g.nu + 255) / 256 < 16 ? (g.nu + 255) / 256 : 16;
  hipLaunchKernelGGL(k_unpermute_rows<R>, dim3(bx, g.nv), dim3(256), 0, st,
                     (const cplx<R>*)src, (cplx<R>*)dst, g);
}

template <typename R>
void launch_screen_bcast(const void* img, int img_real, void* planes,
                         const Geo& g, hipStream_t st) {
  const int64_t npix = (int64_t)g.nu * g.nv;
  hipLaunchKernelGGL(k_screen_bcast<R>, dim3((unsigned)((npix + 255) / 256)),
                     dim3(256), 0, st, img, img_real, (cplx<R>*)planes, g);
}

template <typename R>
void launch_wcorrect(const void* F, void* img, const Geo& g, hipStream_t st) {
  const int64_t npix = (int64_t)g.nu * g.nv;
  hipLaunchKernelGGL(k_wcorrect<R>, dim3((unsigned)((npix + 255) / 256)),
                     dim3(256), 0, st, (const cplx<R>*)F, (cplx<R>*)img, g);
}

template <typename R>
void launch_fill_zero(void* p, int64_t n, hipStream_t st) {
  if (n == 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill_zero<R>, dim3((unsigned)blocks), dim3(256), 0, st,
                     (cplx<R>*)p, n);
}

void launch_zero_u32(uint32_t* p, int64_t n, hipStream_t st) {
  if (n == 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_fill_zero_u32, dim3((unsigned)blocks), dim3(256), 0, st,
                     p, n);
}

template <typename R>
void launch_tables(const Geo& g, void* tw_u, void* tw_v, double* corr,
                   uint32_t* zeros, hipStream_t st) {
  hipLaunchKernelGGL(k_tables<R>, dim3((g.nu + g.nv + 63) / 64), dim3(64), 0,
                     st, g, (cplx<R>*)tw_u, (cplx<R>*)tw_v, corr, zeros);
}

#define WS_INST(R)                                                            \
  template bool launch_fft_rows<R>(void*, int, int64_t, const void*, int,    \
                                   void*, const uint32_t*, int,            \
                                   hipStream_t);                             \
  template bool launch_fft_cols<R>(void*, int, int, int, const void*, int,   \
                                   const uint32_t*, int, const uint32_t*,    \
                                   const void*, const uint32_t*, uint32_t,   \
                                   hipStream_t);                             \
  template bool launch_row_screen_sum<R>(const void*, void*, const Geo&,     \
                                         const void*, const uint32_t*,       \
                                         hipStream_t);                       \
  template bool launch_screen_row_bcast<R>(const void*, int, void*,          \
                                           const Geo&, const void*,          \
                                           hipStream_t);                     \
  template void launch_wcorrect<R>(const void*, void*, const Geo&,           \
                                   hipStream_t);                             \
  template bool launch_fft_cols4<R>(void*, int, int, int, const void*, int,  \
                                    const uint32_t*, int, const uint32_t*,   \
                                    const void*, hipStream_t);               \
  template void launch_unpermute_rows<R>(const void*, void*, const Geo&,     \
                                         hipStream_t);                       \
  template void launch_screen_bcast<R>(const void*, int, void*, const Geo&,  \
                                       hipStream_t);                         \
  template void launch_fill_zero<R>(void*, int64_t, hipStream_t);           \
  template void launch_tables<R>(const Geo&, void*, void*, double*,         \
                                 uint32_t*, hipStream_t);
WS_INST(float)
WS_INST(double)
#undef WS_INST

}  // namespace ws
