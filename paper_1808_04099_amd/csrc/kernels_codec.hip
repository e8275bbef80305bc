// Per-cube lossy wavelet compression of an FP64 cell field (Sec. 6.4.1, Alg. "Compression
// algorithm"): each cube is transformed on its own (CDF 5/3 lifting along x, y and z, log2(n)
// levels, symmetric extension at the cube's faces, coarse half of each axis first), its
// coefficients quantised with one uniform step, and the codes packed in groups of 32 at the
// group's bit width (zigzag map for the sign).  The cubes' streams are concatenated behind a
// header that records where each one starts.  Stream layout (little-endian):
//   0 "BCMW" | 4 version 1 | 8 number of cubes | 12 n | 16 levels | 20 zero | 24 step (FP64)
//   32 cube offsets, (number of cubes + 1) x u64, relative to the data start
//   data: per cube the G = n^3/32 group widths (bytes, zero-padded to 4), then for each group
//   its w 32-bit words, code j at bits j w .. j w + w - 1.
//
// Layout.  A workgroup of 256 lanes takes a unit of CPB = 256 / n^2 cubes (1 at 16^3, 4 at 8^3,
// 16 at 4^3); lane l of a cube's n^2 lanes owns column (i, j) = (l mod n, l / n).  The first
// level lifts lines held in registers, exchanged through LDS between the axes (rows padded by
// one value, so that lanes on x lines hit distinct banks); the remaining levels, one eighth of
// the values, stay inside one wavefront and need no workgroup barrier.  A group of 32 codes is
// a half-wavefront at one k (two planes of a cube at 4^3), so widths are DPP reductions and
// the words are gathered from codes in LDS: the encoder writes packed words, and a second
// kernel moves each cube's words to their place once the sizes are scanned.
//
// What bounds it: on 8192 cubes of 16^3 (268 MB, 54 us at a copy's rate, ratio 1:10) the encoder
// takes 100 us and the decoder 82 us; their VALU work is 41 and 32 us of that and the LDS
// traffic 38 and 36 us, which overlap only in part because every cube alternates between them
// at barriers.  Before, 4-byte codes were written and packed in another pass, the small levels
// ran on whole-workgroup barriers and one lane summed the 128 group widths: 136 + 100 us and
// 187 us.  A compress call went from 267 to 129 us, a decompress call from 257 to 93 us.
//
// The lifting scales by 1/2 and 1/4 (exact), and the quantiser's result is that of an IEEE
// division by the step rounded half to even, so the codes and bytes depend on no operation
// order that another implementation of the same steps could do differently.
#include "kernels.hpp"
#include "tile.hpp"

namespace bcm {

namespace {

// Lifting of one line of M values (M even) in registers, coarse half first.
template <int M>
__device__ __forceinline__ void lift_line(double (&x)[M]) {
  constexpr int H = M / 2;
  double s[H], d[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double right = 2 * i + 2 < M ? x[2 * i + 2 < M ? 2 * i + 2 : 0] : x[M - 2];
    d[i] = x[2 * i + 1] - (x[2 * i] + right) * 0.5;
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double left = i > 0 ? d[i > 0 ? i - 1 : 0] : d[0];
    s[i] = x[2 * i] + (left + d[i]) * 0.25;
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    x[i] = s[i];
    x[H + i] = d[i];
  }
}
template <int M>
__device__ __forceinline__ void unlift_line(double (&x)[M]) {
  constexpr int H = M / 2;
  double e[H], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double left = i > 0 ? x[H + (i > 0 ? i - 1 : 0)] : x[H];
    e[i] = x[i] - (left + x[H + i]) * 0.25;
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const double right = i + 1 < H ? e[i + 1 < H ? i + 1 : 0] : e[H - 1];
    o[i] = x[H + i] + (e[i] + right) * 0.5;
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    x[2 * i] = e[i];
    x[2 * i + 1] = o[i];
  }
}

template <int M>
__device__ __forceinline__ void get_line(double (&x)[M], const double* c, int base, int st) {
#pragma unroll
  for (int q = 0; q < M; ++q) x[q] = c[base + q * st];
}
template <int M>
__device__ __forceinline__ void put_line(const double (&x)[M], double* c, int base, int st) {
#pragma unroll
  for (int q = 0; q < M; ++q) c[base + q * st] = x[q];
}

// Geometry of a unit.  The cube in LDS has each x row padded by one value (row pitch NL + 1):
// lanes lifting x lines read values NL + 1 apart, not NL (a multiple of the bank count).
template <int NL>
struct Wc {
  static constexpr int N2 = NL * NL, N3 = N2 * NL, H = NL / 2;
  static constexpr int CPB = 256 / N2;               // cubes per workgroup
  static constexpr int G = N3 / 32, GP = (G + 3) / 4 * 4;  // groups per cube, width-table bytes
  static constexpr int UG = CPB * G;                 // groups per unit (at most 128)
  static constexpr int UW = UG * 32;                 // words per unit at most
  static constexpr int R = NL + 1, P = NL * R, SIZE = NL * P;
  __device__ static int of(int e) { return e + e / NL; }  // element e = (k NL + j) NL + i
};

// Orders the LDS accesses of one wavefront (the hardware keeps them in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Levels M, M/2, ..., 2 of the corner block of one cube (c: its LDS block), all by the first
// M^2 lanes of the cube, which lie in one wavefront (M <= 8): forward x, y, z per level going
// down, inverse z, y, x per level coming back up.
template <int NL, int M, bool INV>
__device__ __forceinline__ void corner_axis(double* c, int l, int axis) {
  using W = Wc<NL>;
  if (l < M * M) {
    const int a = l % M, b = l / M;
    const int base = axis == 0 ? b * W::P + a * W::R : axis == 1 ? b * W::P + a : b * W::R + a;
    const int st = axis == 0 ? 1 : axis == 1 ? W::R : W::P;
    double x[M];
    get_line<M>(x, c, base, st);
    if (INV)
      unlift_line<M>(x);
    else
      lift_line<M>(x);
    put_line<M>(x, c, base, st);
  }
  wave_sync();
}
template <int NL, int M>
__device__ __forceinline__ void corner_fwd(double* c, int l) {
  if constexpr (M >= 2) {
    for (int ax = 0; ax < 3; ++ax) corner_axis<NL, M, false>(c, l, ax);
    corner_fwd<NL, M / 2>(c, l);
  }
}
template <int NL, int M>
__device__ __forceinline__ void corner_inv(double* c, int l) {
  if constexpr (M >= 2) {
    corner_inv<NL, M / 2>(c, l);
    for (int ax = 2; ax >= 0; --ax) corner_axis<NL, M, true>(c, l, ax);
  }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((may_alias)) u32x4_alias;
typedef double double2_8 __attribute__((ext_vector_type(2), aligned(8)));

constexpr uint32_t kWcMagic = 0x574D4342u;           // "BCMW"
constexpr unsigned long long kWcBad = 1ull << 63;    // mark of a cube in the size array

__device__ __forceinline__ int bit_length(uint32_t v) { return v ? 32 - __clz(v) : 0; }

// OR over rows of 16 lanes (valid on the last lane of each row), then over half-wavefronts
// (valid on lanes 31 and 63).
__device__ __forceinline__ uint32_t or_row(uint32_t v) {
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xf, 0xf, true));  // row_shr 1
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xf, 0xf, true));
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xf, 0xf, true));
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xf, 0xf, true));
  return v;
}
__device__ __forceinline__ uint32_t or_half(uint32_t v) {
  v = or_row(v);
  v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xa, 0xf, false));  // row_bcast 15
  return v;
}

// Exclusive prefix of the unit's group widths (n <= 128), by the first wavefront: pre[0..n],
// each with its group's width in the low 6 bits.
__device__ __forceinline__ void scan_widths(const int* wid, int* pre, int n) {
  if (threadIdx.x >= 64) return;
  const int t = threadIdx.x;
  const int w0 = 2 * t < n ? wid[2 * t] : 0, w1 = 2 * t + 1 < n ? wid[2 * t + 1] : 0;
  int s = w0 + w1;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(s, o, 64);
    if (t >= o) s += up;
  }
  const int ex = s - w0 - w1;
  if (2 * t < n) pre[2 * t] = ex << 6 | w0;
  if (2 * t + 1 < n) pre[2 * t + 1] = (ex + w0) << 6 | w1;
  if (t == 63) pre[n] = s << 6;
}

// Transform, quantise and pack: each cube's group widths, words (at its place in a.words) and
// stream size.
template <int NL>
__global__ __launch_bounds__(256, 4) void k_wc_encode(CodecArgs a) {
  using W = Wc<NL>;
  __shared__ __align__(16) double c[W::CPB * W::SIZE];
  __shared__ int wid[W::UG];
  __shared__ int pre[W::UG + 1];
  __shared__ int bad[W::CPB];
  u32x4_alias* zero4 = reinterpret_cast<u32x4_alias*>(c);
  u32_alias* words = reinterpret_cast<u32_alias*>(c);  // once the coefficients are in registers
  static_assert(sizeof(c) >= size_t(W::UW) * 4, "the words of a unit fit in the cube's LDS block");
  // (one cube per unit at 16^3: s is then a constant, and the cube and its pointers scalar)
  const int t = threadIdx.x, s = W::CPB == 1 ? 0 : t / W::N2, l = W::CPB == 1 ? t : t % W::N2;
  const int units = (a.n_cubes + W::CPB - 1) / W::CPB;
  const bool exact = !(a.step > 1e-290 && a.step < 1e290);
  const double inv = 1.0 / a.step;
  double* cs = c + s * W::SIZE;
  for (int u = blockIdx.x, turn = blockIdx.x >> 3; u < units; u += gridDim.x, ++turn) {
    const int cube = u * W::CPB + s;
    const bool live = cube < a.n_cubes;
    int lu = l;  // opaque: LDS addresses are recomputed per unit, not all held in registers
    asm volatile("" : "+v"(lu));
    const int i = lu % NL, j = lu / NL;
    // the lane's x line at (y, z) = (i, j), 16 bytes a load; not loaded ahead: four workgroups
    // a CU hide the wait better than 32 registers of prefetch, which spilled (131 us a call
    // against 152)
    double x[NL];
    const double2_8* src = reinterpret_cast<const double2_8*>(a.field + (size_t)(live ? cube : 0) * W::N3 + lu * NL);
#pragma unroll
    for (int r = 0; r < NL / 2; ++r) {
      const double2_8 v = src[r];
      x[2 * r] = live ? v[0] : 0.0;
      x[2 * r + 1] = live ? v[1] : 0.0;
    }
    lift_line<NL>(x);
    put_line<NL>(x, cs, j * W::P + i * W::R, 1);
    __syncthreads();
    get_line<NL>(x, cs, j * W::P + i, W::R);  // y line at (x, z) = (i, j)
    lift_line<NL>(x);
    put_line<NL>(x, cs, j * W::P + i, W::R);
    __syncthreads();
    get_line<NL>(x, cs, j * W::R + i, W::P);  // z line at (x, y) = (i, j)
    lift_line<NL>(x);
    if (i < W::H && j < W::H) {
#pragma unroll
      for (int k = 0; k < W::H; ++k) cs[k * W::P + j * W::R + i] = x[k];
    }
    if (l == 0) bad[s] = 0;
    __syncthreads();
    // (the wavefront that takes the corner changes from cube to cube: wavefronts of the same
    // number share a SIMD)
    corner_fwd<NL, W::H>(cs, NL == 16 ? (t + 64 * turn) & 255 : l);
    __syncthreads();
    if (i < W::H && j < W::H) {
#pragma unroll
      for (int k = 0; k < W::H; ++k) x[k] = cs[k * W::P + j * W::R + i];
    }
    // Codes: rint(v / step) of the IEEE quotient.  v * inv differs from the quotient by less
    // than 2^-51 of it, so the two round to the same integer unless a half-integer lies that
    // close; a wavefront with such a value (or one that is not finite) takes the division.
    uint32_t z[NL];
    double top = 0.0;
    bool near = exact;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const double q = x[k] * inv, r = rint(q);
      near |= !(fabs(q - r) <= 0.5 - fabs(q) * 0x1p-50);
      top = fmax(top, fabs(r));
      const int qi = int(r);
      z[k] = (uint32_t(qi) << 1) ^ uint32_t(qi >> 31);
    }
    if (__any(near || !(top < 1073741824.0))) {
      bool over = false;
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const double r = rint(x[k] / a.step);
        const bool fits = fabs(r) < 1073741824.0;  // 2^30; false for NaN
        over |= !fits;
        const int qi = fits ? int(r) : 0;
        z[k] = (uint32_t(qi) << 1) ^ uint32_t(qi >> 31);
      }
      if (over) bad[s] = 1;
    }
    if constexpr (NL >= 8) {
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const uint32_t m = or_half(z[k]);
        if ((t & 31) == 31) wid[s * W::G + k * (W::N2 / 32) + (l >> 5)] = bit_length(m);
      }
    } else {
#pragma unroll
      for (int k = 0; k < NL; k += 2) {
        const uint32_t m = or_row(z[k] | z[k + 1]);
        if ((t & 15) == 15) wid[s * W::G + (k >> 1)] = bit_length(m);
      }
    }
    __syncthreads();
    scan_widths(wid, pre, W::UG);
#pragma unroll
    for (int r = 0; r < W::UW / 1024; ++r) zero4[r * 256 + t] = u32x4{0, 0, 0, 0};
    __syncthreads();
    // each code is ORed into its one or two words
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int e = k * W::N2 + l, pw = pre[s * W::G + (e >> 5)], w = pw & 63;
      const int bit = (pw >> 6) * 32 + (e & 31) * w, sh = bit & 31;
      if (z[k]) {
        const uint64_t v = uint64_t(z[k]) << sh;
        __hip_atomic_fetch_or(words + (bit >> 5), uint32_t(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (v >> 32)
          __hip_atomic_fetch_or(words + (bit >> 5) + 1, uint32_t(v >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
    const int first = pre[s * W::G] >> 6, count = (pre[(s + 1) * W::G] >> 6) - first;
    if (live) {
      for (int q = l; q < count; q += W::N2) a.words[(size_t)cube * W::N3 + q] = words[first + q];
      if (l < W::G) a.widths[(size_t)cube * W::G + l] = uint8_t(wid[s * W::G + l]);
      if (l == 0) a.sizes[cube] = (unsigned long long)(W::GP + 4 * count) | (bad[s] ? kWcBad : 0);
    }
    __syncthreads();
  }
}

// The verdict of a call to the workspace and to the pinned host mirror (if any), as the bits of
// two scalars.
__device__ __forceinline__ void wc_publish(const CodecArgs& a, unsigned long long total, unsigned long long flags) {
  a.result[0] = total;
  a.result[1] = flags;
  if (a.mirror) {
    a.mirror->sc.spare[0] = __longlong_as_double((long long)total);
    a.mirror->sc.spare[1] = __longlong_as_double((long long)flags);
    __threadfence_system();
    __hip_atomic_store(&a.mirror->seq, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Header and cube offsets: one workgroup scans the cube sizes, eight per lane and round.  The total and the verdict
// (kWcOver: a code too large; kWcFull: the buffer too small) are published here, so that the
// host learns them while the words are still being moved; k_wc_pack moves nothing unless the
// verdict is 0.
__global__ __launch_bounds__(1024) void k_wc_header(CodecArgs a) {
  __shared__ unsigned long long wave[2][16];
  unsigned char* h = static_cast<unsigned char*>(a.stream);
  unsigned long long* offs = reinterpret_cast<unsigned long long*>(h + 32);
  const int t = threadIdx.x;
  constexpr int PER = 8;  // sizes per lane and round, all loaded before any is used
  unsigned long long total = 0, marks = 0;
  int buf = 0;
  for (int base = 0; base < a.n_cubes; base += 1024 * PER, buf ^= 1) {
    const int e0 = base + t * PER;
    unsigned long long v[PER], sum = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r) v[r] = e0 + r < a.n_cubes ? a.sizes[e0 + r] : 0ull;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      marks |= v[r];
      v[r] &= ~kWcBad;
      sum += v[r];
    }
    unsigned long long s = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long up = __shfl_up(s, o, 64);
      if ((t & 63) >= o) s += up;
    }
    if ((t & 63) == 63) wave[buf][t >> 6] = s;
    __syncthreads();  // (two buffers: the next round's writes cannot overtake these reads)
    unsigned long long at = total + s - sum;
    for (int w = 0; w < 16; ++w) {
      if (w < (t >> 6)) at += wave[buf][w];
      total += wave[buf][w];
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      if (e0 + r < a.n_cubes) offs[e0 + r] = at;
      at += v[r];
    }
  }
  const bool over = __syncthreads_or((marks & kWcBad) != 0);
  if (t == 0) {
    const uint32_t head[6] = {kWcMagic, 1u, uint32_t(a.n_cubes), uint32_t(a.n), uint32_t(a.levels), 0u};
    for (int q = 0; q < 6; ++q) reinterpret_cast<uint32_t*>(h)[q] = head[q];
    *reinterpret_cast<double*>(h + 24) = a.step;
    offs[a.n_cubes] = total;
    const bool full = 32 + 8 * (unsigned long long)(a.n_cubes + 1) + total > a.capacity;
    wc_publish(a, total, (over ? kWcOver : 0) | (full ? kWcFull : 0));
  }
}

// Widths and words of every cube to its offset: one wavefront per cube.
template <int NL>
__global__ __launch_bounds__(256) void k_wc_pack(CodecArgs a) {
  using W = Wc<NL>;
  unsigned char* h = static_cast<unsigned char*>(a.stream);
  const unsigned long long* offs = reinterpret_cast<const unsigned long long*>(h + 32);
  unsigned char* data = h + 32 + 8 * (size_t)(a.n_cubes + 1);
  const int l = threadIdx.x & 63;
  if (a.result[1] != 0) return;
  for (int cube = blockIdx.x * 4 + (threadIdx.x >> 6); cube < a.n_cubes; cube += gridDim.x * 4) {
    const unsigned long long o0 = offs[cube], o1 = offs[cube + 1];
    const int words = int((o1 - o0 - W::GP) / 4);
    uint32_t* out = reinterpret_cast<uint32_t*>(data + o0);
    if (l < W::GP / 4) {  // width table, four bytes per word
      uint32_t v = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int g = 4 * l + b;
        v |= uint32_t(g < W::G ? a.widths[(size_t)cube * W::G + g] : 0) << (8 * b);
      }
      out[l] = v;
    }
    const uint32_t* src = a.words + (size_t)cube * W::N3;
    out += W::GP / 4;
#pragma unroll 4
    for (int q = l; q < words; q += 64) out[q] = src[q];
  }
}

// Whether a stream's header belongs to this mesh and its last offset to the stream's length.
__device__ __forceinline__ bool wc_header_ok(const CodecArgs& a, double& step) {
  const unsigned char* h = static_cast<const unsigned char*>(a.stream_in);
  const uint32_t* hw = reinterpret_cast<const uint32_t*>(h);
  step = *reinterpret_cast<const double*>(h + 24);
  return hw[0] == kWcMagic && hw[1] == 1u && int(hw[2]) == a.n_cubes && int(hw[3]) == a.n &&
         int(hw[4]) == a.levels && step > 0.0 && isfinite(step) &&
         reinterpret_cast<const unsigned long long*>(h + 32)[a.n_cubes] == a.data_bytes;
}

// The verdict on a decoded stream from the header and the cubes' marks.
__global__ __launch_bounds__(1024) void k_wc_verdict(CodecArgs a) {
  double step;
  const bool ok = wc_header_ok(a, step);
  unsigned long long marks = 0;
  if (ok)
    for (int e = threadIdx.x; e < a.n_cubes; e += 1024) marks |= a.sizes[e];
  const bool any = __syncthreads_or(marks != 0);
  if (threadIdx.x == 0) wc_publish(a, 0, !ok ? kWcHeader : any ? kWcCube : 0);
}

// Decode: unpack, dequantise, inverse transform.  Nothing is written for a foreign header.
template <int NL>
__global__ __launch_bounds__(256, 4) void k_wc_decode(CodecArgs a) {
  using W = Wc<NL>;
  __shared__ __align__(16) double c[W::CPB * W::SIZE];
  __shared__ int wid[W::UG];
  __shared__ int pre[W::UG + 1];
  __shared__ int bad[W::CPB];
  static_assert(sizeof(c) >= size_t(W::UW) * 4 + 8, "the words of a unit fit in the cube's LDS block");
  u32_alias* words = reinterpret_cast<u32_alias*>(c);  // until the codes are in registers
  const unsigned char* h = static_cast<const unsigned char*>(a.stream_in);
  const unsigned long long* offs = reinterpret_cast<const unsigned long long*>(h + 32);
  const unsigned char* data = h + 32 + 8 * (size_t)(a.n_cubes + 1);
  // (one cube per unit at 16^3: s is then a constant, and the cube and its pointers scalar)
  const int t = threadIdx.x, s = W::CPB == 1 ? 0 : t / W::N2, l = W::CPB == 1 ? t : t % W::N2;
  const int units = (a.n_cubes + W::CPB - 1) / W::CPB;
  double* cs = c + s * W::SIZE;
  double step;
  if (!wc_header_ok(a, step)) return;
  for (int u = blockIdx.x, turn = blockIdx.x >> 3; u < units; u += gridDim.x, ++turn) {
    const int cube = u * W::CPB + s;
    const bool live = cube < a.n_cubes;
    int lu = l;  // opaque: LDS addresses are recomputed per unit, not all held in registers
    asm volatile("" : "+v"(lu));
    const int i = lu % NL, j = lu / NL;
    const unsigned long long o0 = live ? offs[cube] : 0, o1 = live ? offs[cube + 1] : 0;
    const bool room = live && o1 >= o0 && o1 - o0 >= (unsigned long long)W::GP && o1 <= a.data_bytes;
    const uint32_t* in = reinterpret_cast<const uint32_t*>(data + (room ? o0 : 0));
    if (l == 0) bad[s] = live && !room;
    __syncthreads();
    if (l < W::G) {
      const int w = room ? int(in[l >> 2] >> (8 * (l & 3)) & 0xFFu) : 0;
      if (w > 32) bad[s] = 1;
      wid[s * W::G + l] = w > 32 ? 0 : w;
    }
    __syncthreads();
    scan_widths(wid, pre, W::UG);
    __syncthreads();
    const int first = pre[s * W::G] >> 6, count = (pre[(s + 1) * W::G] >> 6) - first;
    const bool valid = room && !bad[s] && o1 - o0 == (unsigned long long)W::GP + 4ull * count;
    if (live && l == 0) a.sizes[cube] = valid ? 0 : kWcBad;  // an invalid cube decodes to zeros
    if (valid)
      for (int q = l; q < count; q += W::N2) words[first + q] = in[W::GP / 4 + q];
    __syncthreads();
    double x[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int e = k * W::N2 + l, pw = pre[s * W::G + (e >> 5)], w = valid ? pw & 63 : 0;
      const int bit = (pw >> 6) * 32 + (e & 31) * w, wi = bit >> 5;
      // (the second word may be the next group's or unwritten: its bits are masked off)
      const uint32_t z = __builtin_amdgcn_alignbit(words[wi + 1], words[wi], bit & 31) &
                         (w ? 0xFFFFFFFFu >> (32 - w) : 0u);
      x[k] = double(int(z >> 1) ^ -int(z & 1)) * step;
      if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (else every k's LDS reads are live at once)
    }
    __syncthreads();
    if (i < W::H && j < W::H) {
#pragma unroll
      for (int k = 0; k < W::H; ++k) cs[k * W::P + j * W::R + i] = x[k];
    }
    __syncthreads();
    corner_inv<NL, W::H>(cs, NL == 16 ? (t + 64 * turn) & 255 : l);
    __syncthreads();
    if (i < W::H && j < W::H) {
#pragma unroll
      for (int k = 0; k < W::H; ++k) x[k] = cs[k * W::P + j * W::R + i];
    }
    unlift_line<NL>(x);  // z line at (x, y) = (i, j)
    put_line<NL>(x, cs, j * W::R + i, W::P);
    __syncthreads();
    get_line<NL>(x, cs, j * W::P + i, W::R);  // y line at (x, z) = (i, j)
    unlift_line<NL>(x);
    put_line<NL>(x, cs, j * W::P + i, W::R);
    __syncthreads();
    get_line<NL>(x, cs, j * W::P + i * W::R, 1);  // x line at (y, z) = (i, j)
    unlift_line<NL>(x);
    put_line<NL>(x, cs, j * W::P + i * W::R, 1);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NL; ++r) {
      const int e = r * 256 + t;
      if (W::CPB == 1 || u * W::CPB + e / W::N3 < a.n_cubes)
        st_nt(a.field_out + (size_t)u * (256 * NL) + e, c[e / W::N3 * W::SIZE + W::of(e % W::N3)]);
    }
    __syncthreads();
  }
}

}  // namespace

#define BCM_WC_NL(NLV, CALL)                          \
  switch (NLV) {                                      \
    case 16: { constexpr int NLC = 16; CALL; } break; \
    case 8: { constexpr int NLC = 8; CALL; } break;   \
    case 4: { constexpr int NLC = 4; CALL; } break;   \
    default: return hipErrorInvalidValue;             \
  }

hipError_t launch_wc_encode(int NL, const CodecArgs& a, int grid, hipStream_t s) {
  BCM_WC_NL(NL, hipLaunchKernelGGL((k_wc_encode<NLC>), dim3(grid), dim3(256), 0, s, a));
  return hipGetLastError();
}
hipError_t launch_wc_header(const CodecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_wc_header, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_wc_pack(int NL, const CodecArgs& a, int grid, hipStream_t s) {
  BCM_WC_NL(NL, hipLaunchKernelGGL((k_wc_pack<NLC>), dim3(grid), dim3(256), 0, s, a));
  return hipGetLastError();
}
hipError_t launch_wc_decode(int NL, const CodecArgs& a, int grid, hipStream_t s) {
  BCM_WC_NL(NL, hipLaunchKernelGGL((k_wc_decode<NLC>), dim3(grid), dim3(256), 0, s, a));
  return hipGetLastError();
}
hipError_t launch_wc_verdict(const CodecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_wc_verdict, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}

}  // namespace bcm
