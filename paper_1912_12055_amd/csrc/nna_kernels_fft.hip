// The STFT and Mel transforms of plain DFT bins with fixed kernels as a fast Fourier transform per frame.
//
// eq. (DFT2)'s kernels are w[n] e^{-2 pi i k n / N}: one frame's N/2 + 1 bins are the DFT of the windowed frame, and the
// sums over n can be taken in stages.  The real frame is packed into M = N/2 complex values z[m] = x[2m] + i x[2m+1], a
// complex DFT of M points is taken in two or three passes of radix 4 / 8 / 16, and the bins follow from
// X[k] = (Z[k] + conj Z[M-k]) / 2 - i e^{-2 pi i k / N} (Z[k] - conj Z[M-k]) / 2.  About 60,000 operations per frame of
// 2,048 samples instead of 2.1 million in the contraction that used every symmetry of its kernels.
//
// A wave owns whole frames up to N = 2,048, so the passes exchange their values through LDS without a barrier (a wave's LDS
// accesses complete in order); real and imaginary parts go one after the other through the same words.  The region a frame
// exchanges through is the row of the output tile its finished bins are written to.  The tile turns bins-per-frame into runs
// of consecutive frames of one bin, the order of the output; while one tile is computed, the one before it is written out (where LDS
// holds two tiles of more than two frames: launch_fixed).
//
// What bounds it: two waves per SIMD (the tables a lane keeps in registers), a chain of passes through LDS each.  Without its
// output the call below takes 0.82 ms, the vector ALUs' time; meeting once a tile and the stores' own instructions add the rest.
//
// 1,770 x 176,400 samples, N = 2,048, hop 512 (MI355X): magnitudes 10.1 ms contracted, 2.20 with a tile computed, then stored
// between two barriers and neighbouring tiles 29 us apart, 1.51 with samples requested word by word, now 1.35 (either way 3.66 GB are written for
// 2.50: runs of half a line; writing them so, with nothing computed, takes 1.38 by itself, in runs that begin at 64 bytes 0.83);
// N = 1,024, hop 256, complex: 4.02 -> 2.35.  Mel, 64 x 110,250, 128 bands: 808 us contracted, 48 -> 39 -> 37; 1,770 x 80,000,
// N = 4,096, 512 bands: 34.9 ms, 2.02 -> 1.72 -> 1.53.  4 x 22,050: 300 -> 10 us.  Tried: window and twiddles read from the caches for
// every frame with four waves per SIMD (2.85 ms: the vector memory path saturates), from LDS with four waves per SIMD (spills,
// 1.87 ms), three waves per SIMD (spills, 4.3 ms), the tile stored by two workgroups of four waves (runs of 32 bytes, 2.04 ms),
// frames in a ring from which every row is written in segments that begin at 64 bytes (2.7 GB written, but waves that meet every step: 1.47 ms).
#include "nna_device.h"

namespace nna {
namespace {

// two samples at any word
typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));

__device__ __forceinline__ void wave_fence() {
  // orders the LDS accesses of one wave for the compiler; the hardware keeps them in order by itself
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

struct cplx {
  float x, y;
};
__device__ __forceinline__ cplx operator+(cplx a, cplx b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cplx operator-(cplx a, cplx b) { return {a.x - b.x, a.y - b.y}; }
// a * (c - i s): twiddles are stored as (cos, sin) of the positive angle
__device__ __forceinline__ cplx twiddle(cplx a, float2 w) {
  return {__builtin_fmaf(a.y, w.y, a.x * w.x), __builtin_fmaf(-a.x, w.y, a.y * w.x)};
}
__device__ __forceinline__ cplx minus_i(cplx a) { return {a.y, -a.x}; }

// DFTs of 2 .. 16 points in registers, natural order in and out
template <int R>
__device__ __forceinline__ void dft(cplx (&a)[R]);

template <>
__device__ __forceinline__ void dft<2>(cplx (&a)[2]) {
  const cplx s = a[0] + a[1], d = a[0] - a[1];
  a[0] = s;
  a[1] = d;
}
__device__ __forceinline__ void dft4(cplx& a0, cplx& a1, cplx& a2, cplx& a3) {
  const cplx t0 = a0 + a2, t1 = a0 - a2, t2 = a1 + a3, t3 = minus_i(a1 - a3);
  a0 = t0 + t2;
  a1 = t1 + t3;
  a2 = t0 - t2;
  a3 = t1 - t3;
}
template <>
__device__ __forceinline__ void dft<4>(cplx (&a)[4]) {
  dft4(a[0], a[1], a[2], a[3]);
}
template <>
__device__ __forceinline__ void dft<8>(cplx (&a)[8]) {
  constexpr float r = 0.70710678118654752440f;
  dft4(a[0], a[2], a[4], a[6]);
  dft4(a[1], a[3], a[5], a[7]);
  const cplx o0 = a[1], o1 = {(a[3].x + a[3].y) * r, (a[3].y - a[3].x) * r}, o2 = minus_i(a[5]),
             o3 = {(a[7].y - a[7].x) * r, -(a[7].x + a[7].y) * r};
  const cplx e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
  a[0] = e0 + o0;
  a[1] = e1 + o1;
  a[2] = e2 + o2;
  a[3] = e3 + o3;
  a[4] = e0 - o0;
  a[5] = e1 - o1;
  a[6] = e2 - o2;
  a[7] = e3 - o3;
}
template <>
__device__ __forceinline__ void dft<16>(cplx (&a)[16]) {
  constexpr float r = 0.70710678118654752440f, c1 = 0.92387953251128675613f, s1 = 0.38268343236508977173f;
#pragma unroll
  for (int n = 0; n < 4; ++n) dft4(a[n], a[n + 4], a[n + 8], a[n + 12]);
  // a[n + 4 k] times e^{-2 pi i n k / 16}
  a[5] = twiddle(a[5], float2{c1, s1});
  a[9] = {(a[9].x + a[9].y) * r, (a[9].y - a[9].x) * r};
  a[13] = twiddle(a[13], float2{s1, c1});
  a[6] = {(a[6].x + a[6].y) * r, (a[6].y - a[6].x) * r};
  a[10] = minus_i(a[10]);
  a[14] = {(a[14].y - a[14].x) * r, -(a[14].x + a[14].y) * r};
  a[7] = twiddle(a[7], float2{s1, c1});
  a[11] = {(a[11].y - a[11].x) * r, -(a[11].x + a[11].y) * r};
  a[15] = twiddle(a[15], float2{-c1, -s1});
#pragma unroll
  for (int k = 0; k < 4; ++k) dft4(a[4 * k], a[4 * k + 1], a[4 * k + 2], a[4 * k + 3]);
  // a[4 k + m] holds bin k + 4 m
  cplx b[16];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int m = 0; m < 4; ++m) b[k + 4 * m] = a[4 * k + m];
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = b[i];
}
// odd radices of the general kernel, from the definition with the terms r and R - r taken together
template <int R>
__device__ __forceinline__ void dft_odd(cplx (&a)[R]) {
  constexpr float pi2 = 6.28318530717958647693f;
  constexpr int H = R / 2;
  cplx s[H], d[H], y[R];
  cplx sum = a[0];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    s[i] = a[i + 1] + a[R - 1 - i];
    d[i] = a[i + 1] - a[R - 1 - i];
    sum = sum + s[i];
  }
  y[0] = sum;
#pragma unroll
  for (int k = 1; k <= H; ++k) {
    cplx c = a[0], e = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int m = (k * (i + 1)) % R;
      const float cs = __builtin_cosf(pi2 * m / R), sn = __builtin_sinf(pi2 * m / R);  // constants after unrolling
      c = {__builtin_fmaf(s[i].x, cs, c.x), __builtin_fmaf(s[i].y, cs, c.y)};
      e = {__builtin_fmaf(d[i].x, sn, e.x), __builtin_fmaf(d[i].y, sn, e.y)};
    }
    // y[k] = c - i e, y[R - k] = c + i e
    y[k] = {c.x + e.y, c.y - e.x};
    y[R - k] = {c.x - e.y, c.y + e.x};
  }
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = y[i];
}
template <>
__device__ __forceinline__ void dft<3>(cplx (&a)[3]) {
  dft_odd<3>(a);
}
template <>
__device__ __forceinline__ void dft<5>(cplx (&a)[5]) {
  dft_odd<5>(a);
}
template <>
__device__ __forceinline__ void dft<7>(cplx (&a)[7]) {
  dft_odd<7>(a);
}

// bins k and M - k from Z[k] and Z[M - k]; w = (cos, sin)(2 pi k / N); the factor 1/2 is in the window
__device__ __forceinline__ void split_pair(cplx zk, cplx zm, float2 w, cplx& xk, cplx& xm) {
  const cplx e = {zk.x + zm.x, zk.y - zm.y};
  const cplx p = twiddle(cplx{zk.y + zm.y, zm.x - zk.x}, w);
  xk = {e.x + p.x, e.y + p.y};
  xm = {e.x - p.x, p.y - e.y};
}

// Frame `fi` of the tile that starts at frame t0 of waveform b0
__device__ __forceinline__ void frame_of(int fi, long long b0, int t0, int T, long long& b, int& t) {
  const int u = t0 + fi, q = u < T ? 0 : u / T;
  b = b0 + q;
  t = u - q * T;
}

__device__ __forceinline__ int reflect(int i, int L) { return i < 0 ? -i : (i >= L ? 2 * (L - 1) - i : i); }

template <int FMT>
__device__ __forceinline__ float formatted(const float* __restrict__ row, int r, int plane) {
  if constexpr (FMT == NNA_OUT_PHASE)
    return atan2f(row[plane + r], row[r]);
  else if constexpr (FMT == NNA_OUT_COMPLEX)
    return row[(r & 1) * plane + (r >> 1)];
  else if constexpr (FMT == NNA_OUT_MAGNITUDE)
    return __builtin_amdgcn_sqrtf(row[r]);
  else
    return FMT == NNA_OUT_POWER ? row[r] : logf(fmaxf(row[r], 1e-10f));
}

// The finished tile, frame after frame in LDS, to [waveform][row][frame]: a wave writes G = 64 / TF rows per instruction,
// TF consecutive frames each.  The G rows lie TF apart, which spreads their LDS reads over all banks (the pitch is odd).
// Part `part` of 2^lg_parts of this wave's share, a run of consecutive rows: constant steps in LDS, a scalar step in memory.
template <int FMT>
__device__ __forceinline__ void store_rows(const float* __restrict__ tile, int pitch, int plane, int lg_tf, int rows,
                                           float* __restrict__ out, long long n_left, long long b0, int t0, int T,
                                           int wave, int n_wave, int lane, int part, int lg_parts) {
  const int TF = 1 << lg_tf, f = lane & (TF - 1), r_lane = (lane >> lg_tf) << lg_tf;
  if (f >= n_left) return;
  long long b;
  int t;
  frame_of(f, b0, t0, T, b, t);
  float* __restrict__ op = out + (b * rows + r_lane) * (long long)T + t;
  // (complex: an odd r_lane only where TF is 1, and then every r below is even)
  const float* __restrict__ row = tile + f * pitch + (FMT == NNA_OUT_COMPLEX ? (r_lane & 1) * plane + r_lane / 2 : r_lane);
  const int full = rows >> 6 << lg_tf;  // instructions that write G rows
  int v = full * wave / n_wave, v_end = full * (wave + 1) / n_wave;
  const int n = v_end - v;
  v_end = v + (n * (part + 1) >> lg_parts);
  v += n * part >> lg_parts;
  // Fewer than eight frames: four rows at a time.  One after the other, each waiting for its own word, 4 x 22,050 samples, complex, take
  // 12.0 us instead of 10.4.  Rows of two frames do better one by one where the chip is full (865 frames of 4,096, complex: 23.6 us, 24.6 by
  // fours), but for phases (173 frames: 13.6, 12.5).
  if (TF < 8 && (TF != 2 || FMT == NNA_OUT_PHASE))
#pragma unroll 1
    for (; v + 4 <= v_end; v += 4) {
      float x[4];
      auto row_of = [&](int i) { return ((v + i) >> lg_tf << 6) + ((v + i) & (TF - 1)); };
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = formatted<FMT>(row, row_of(i), plane);
#pragma unroll
      for (int i = 0; i < 4; ++i) op[(long long)row_of(i) * T] = x[i];
    }
  while (v < v_end) {
    const int r = ((v >> lg_tf) << 6) + (v & (TF - 1));
    if (v + 8 <= v_end && (v & (TF - 1)) + 8 <= TF && (FMT != NNA_OUT_COMPLEX || r % 2 == 0)) {
      const float* __restrict__ src = row + (FMT == NNA_OUT_COMPLEX ? r / 2 : r);
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = formatted<FMT>(src, i, plane);
#pragma unroll
      for (int i = 0; i < 8; ++i) op[(long long)(r + i) * T] = x[i];
      v += 8;
    } else {
      op[(long long)r * T] = formatted<FMT>(row, r, plane);
      ++v;
    }
  }
  // the rows behind the last 64: TF of them per turn, the lanes past the last one idle
  if (part + 1 == 1 << lg_parts)
    for (int i = wave; i < TF && i < (rows & 63); i += n_wave) {
      const int r = (rows & ~63) + i;
      if (r + r_lane < rows) op[(long long)r * T] = formatted<FMT>(row, r, plane);
    }
}

template <int MODE>
__device__ __forceinline__ void store_tile(const float* __restrict__ tile, int pitch, int plane, int lg_tf, int rows,
                                           float* __restrict__ out, int fmt, long long n_left, long long b0, int t0, int T,
                                           int wave, int n_wave, int lane, int part, int lg_parts) {
  if constexpr (MODE == FFT_MODE_CPLX) {
    if (fmt == NNA_OUT_COMPLEX)
      store_rows<NNA_OUT_COMPLEX>(tile, pitch, plane, lg_tf, rows, out, n_left, b0, t0, T, wave, n_wave, lane, part, lg_parts);
    else
      store_rows<NNA_OUT_PHASE>(tile, pitch, plane, lg_tf, rows, out, n_left, b0, t0, T, wave, n_wave, lane, part, lg_parts);
  } else if constexpr (MODE == FFT_MODE_MEL) {
    store_rows<NNA_OUT_POWER>(tile, pitch, plane, lg_tf, rows, out, n_left, b0, t0, T, wave, n_wave, lane, part, lg_parts);
  } else {
    if (fmt == NNA_OUT_MAGNITUDE)
      store_rows<NNA_OUT_MAGNITUDE>(tile, pitch, plane, lg_tf, rows, out, n_left, b0, t0, T, wave, n_wave, lane, part, lg_parts);
    else if (fmt == NNA_OUT_POWER)
      store_rows<NNA_OUT_POWER>(tile, pitch, plane, lg_tf, rows, out, n_left, b0, t0, T, wave, n_wave, lane, part, lg_parts);
    else
      store_rows<NNA_OUT_LOG>(tile, pitch, plane, lg_tf, rows, out, n_left, b0, t0, T, wave, n_wave, lane, part, lg_parts);
  }
}

// Mel bands of the tile: lanes are (band, frame), so the frames of one band share its weights and a wave's LDS reads
// are runs of TF words.  Only a band's own bins are visited, four at a time (padded with zero weights).  `mel`, `melw`: the
// tables, in LDS where they fit beside the tile (every band's reads of its descriptor and weights are a chain that the caches
// answer in hundreds of cycles a link).  Bands grow longer upwards: the waves take turns in alternating order.
__device__ __forceinline__ void mel_tile(const FftParams& P, const int4* mel, const float4* melw, const float* __restrict__ tile, int pitch,
                                         int lg_tf, long long n_left, long long b0, int t0, int wave, int n_wave, int lane, int part,
                                         int lg_parts) {
  const int TF = 1 << lg_tf, f = lane & (TF - 1), G = 64 >> lg_tf;
  if (f >= n_left) return;
  long long b;
  int t;
  frame_of(f, b0, t0, P.g.T, b, t);
  float* __restrict__ op = P.out + (b * P.n_mels) * (long long)P.g.T + t;
  const int rounds = (P.n_mels + G * n_wave - 1) / (G * n_wave);
  for (int j = rounds * part >> lg_parts; j < rounds * (part + 1) >> lg_parts; ++j) {
    const int m = (j * n_wave + (j & 1 ? n_wave - 1 - wave : wave)) * G + (lane >> lg_tf);
    if (m >= P.n_mels) continue;
    const int4 d = mel[m];  // first bin, quads of bins, first quad of weights
    const float* __restrict__ p = tile + f * pitch + d.x;
    const float4* w = melw + d.z;
    float a0 = 0.f, a1 = 0.f;
#pragma unroll 2
    for (int i = 0; i < d.y; ++i) {
      const float4 q = w[i];
      a0 = __builtin_fmaf(q.x, p[4 * i], a0);
      a1 = __builtin_fmaf(q.y, p[4 * i + 1], a1);
      a0 = __builtin_fmaf(q.z, p[4 * i + 2], a0);
      a1 = __builtin_fmaf(q.w, p[4 * i + 3], a1);
    }
    op[(long long)m * P.g.T] = a0 + a1;
  }
}

// ---------------------------------------------------------------------------------------
// N = 2 M a power of two, 64 .. 4,096: radices R1, R2 (, R3), V complex values per lane.
// ---------------------------------------------------------------------------------------
constexpr int kLdsTwo = 80 * 1024;   // two workgroups per CU
constexpr int kLdsMax = 156 * 1024;  // one
constexpr int kLdsAll = 160 * 1024;  // ... to the last byte

template <int M, int R1, int R2, int R3, int V, int MODE>
struct FftTile {
  static constexpr int RL = R3 > 1 ? R3 : R2;           // radix of the last pass
  static constexpr int H = M / RL;                      // its butterflies per frame
  static constexpr int TPF = M / V;                     // lanes per frame
  static constexpr int NBL = V / RL;                    // butterflies of the last pass per lane, in pairs j, H - j
  static constexpr int PLANE = M + 1;
  static constexpr int WORDS = MODE == FFT_MODE_CPLX ? 2 * M + 2 : (M + M / 16 > M + 4 ? M + M / 16 : M + 4);
  static constexpr int PITCH = WORDS | 1;
  static constexpr int frames_per_step(int n_wave) { return 64 * n_wave / TPF; }
  // What a workgroup may take of a CU: eight waves are all that its registers hold.  In one workgroup they write longer runs of the
  // output; in two, where the output is small (Mel), the two waves of a SIMD wait for nothing of each other's.
  static constexpr int WAVES = MODE != FFT_MODE_MEL && TPF <= 64 && frames_per_step(8) <= 64 && 2 * frames_per_step(8) * PITCH * 4 <= kLdsAll - 16 ? 8 : 4;
  static constexpr int LDS = WAVES == 8 ? kLdsAll : kLdsTwo;
  // steps of the largest tile: what the LDS holds twice, at most 64 frames (the lanes of a store)
  static constexpr int max_steps(int n_wave, int other_bytes) {
    int n = 1;
    while (2 * n * frames_per_step(n_wave) <= 64 && 4 * n * frames_per_step(n_wave) * PITCH * 4 + other_bytes <= LDS) n *= 2;
    return n;
  }
  static_assert(frames_per_step(4) <= 64 && 2 * frames_per_step(4) * PITCH * 4 + 16 <= LDS, "a tile is at most as wide as a wave");
};

// The sizes that have a kernel of their own, and its shape.
template <int M_, int R1_, int R2_, int R3_, int V_>
struct Shape {
  static constexpr int M = M_, R1 = R1_, R2 = R2_, R3 = R3_, V = V_;
  template <int MODE>
  using Tile = FftTile<M, R1, R2, R3, V, MODE>;
};
constexpr int kShapes[] = {32, 64, 128, 256, 512, 1024, 2048};
template <typename Fn>
bool with_shape(int M, Fn&& fn) {
  switch (M) {
    case 32: fn(Shape<32, 8, 4, 1, 8>{}); return true;
    case 64: fn(Shape<64, 8, 8, 1, 16>{}); return true;
    case 128: fn(Shape<128, 16, 8, 1, 16>{}); return true;
    case 256: fn(Shape<256, 8, 8, 4, 16>{}); return true;
    case 512: fn(Shape<512, 8, 8, 8, 16>{}); return true;
    case 1024: fn(Shape<1024, 16, 16, 4, 16>{}); return true;
    case 2048: fn(Shape<2048, 16, 16, 8, 16>{}); return true;
    default: return false;
  }
}

__device__ __forceinline__ constexpr int padded(int i) { return i + (i >> 4); }  // LDS word of exchanged value i

// WAIT: the samples of frames at a waveform's ends are waited for where they are requested (few_ends).
template <int M, int R1, int R2, int R3, int V, int MODE, bool WAIT>
__global__ __launch_bounds__(512, 2) void fft_kernel(FftParams P) {
  using C = FftTile<M, R1, R2, R3, V, MODE>;
  constexpr int RL = C::RL, H = C::H, TPF = C::TPF, NBL = C::NBL;
  static_assert(R1 * R2 * R3 == M && V % R1 == 0 && V % R2 == 0 && NBL % 2 == 0 && RL % 2 == 0, "pass shape");
  static_assert(R3 == 1 || TPF % R1 == 0, "the middle pass shares one set of twiddles");
  extern __shared__ float tile[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this lane's frame in a step, and its place in the frame
  const int first = TPF >= 64 ? wave / (TPF / 64 > 0 ? TPF / 64 : 1) : wave * (64 / TPF) + lane / TPF;
  const int lt = TPF >= 64 ? (wave % (TPF / 64 > 0 ? TPF / 64 : 1)) * 64 + lane : lane % TPF;
  const int n_wave = blockDim.x >> 6, FPWG = 64 * n_wave / TPF;  // frames per step
  const int TF = 1 << P.lg_tf, L = (int)P.g.L, T = P.g.T;
  const int iters = TF / FPWG;
  // a frame inside one wave needs no barrier between its passes: the wave's LDS accesses complete in order
  auto fence = [] {
    if constexpr (TPF > 64)
      __syncthreads();
    else
      wave_fence();
  };
  // Workgroup ids are dealt round-robin to the 8 XCDs.  An XCD's workgroups take neighbouring tiles at the same time, so that the
  // samples their frames share meet in one L2 while they are there.  (Output lines that a tile begins and its neighbour ends do not: as
  // many bytes are written as with neighbouring tiles one after the other.)
  const long long per_xcd = (P.n_tiles + 7) >> 3, lo = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  const long long hi = ((blockIdx.x & 7) + 1) * per_xcd < P.n_tiles ? ((blockIdx.x & 7) + 1) * per_xcd : P.n_tiles;
  const int stride = gridDim.x >> 3;  // tiles from one of this workgroup's to its next
  if (lo >= hi) return;
  int4* mel = reinterpret_cast<int4*>(tile + P.mel_lds);
  float4* melw = reinterpret_cast<float4*>(mel + P.n_mels);
  if constexpr (MODE == FFT_MODE_MEL) {
    if (P.mel_lds) {  // (every wave is past this when it meets the others at the end of its first tile)
      for (int i = tid; i < P.n_mels; i += blockDim.x) mel[i] = P.mel[i];
      for (int i = tid; i < P.mel_quads; i += blockDim.x) melw[i] = P.melw[i];
    }
  }
  long long b0 = (unsigned long long)(lo << P.lg_tf) / (unsigned)T;  // waveform and frame of the tile's first frame
  int t0 = (int)((lo << P.lg_tf) - b0 * T);
  long long b;  // ... of this lane's next frame
  int t;
  frame_of(first, b0, t0, T, b, t);

  const float2* win = reinterpret_cast<const float2*>(P.win);
  const float2* tw = P.tw;
  // Everything a lane multiplies with stays in its registers: window, twiddles of the middle pass, of the last pass, of the
  // bins.  Read again for every frame (from LDS or the caches) they cost more than the occupancy they leave room for.
  float2 w[V], tl[NBL * (RL - 1)], ts[V / 2];
#pragma unroll
  for (int i = 0; i < V; ++i) w[i] = win[lt + TPF * (i / R1) + (M / R1) * (i % R1)];
  {
    const float4* __restrict__ lt_tw = P.tw_lane + lt;  // lane-ordered: two per load
#pragma unroll
    for (int u = 0; u < NBL * (RL - 1) + V / 2; ++u) {
      const float4 q = lt_tw[u / 2 * TPF];
      (u < NBL * (RL - 1) ? tl[u % (NBL * (RL - 1))] : ts[(u - NBL * (RL - 1)) % (V / 2)]) = u % 2 ? float2{q.z, q.w} : float2{q.x, q.y};
    }
  }
  auto j_last = [&](int i) {  // butterfly i of this lane in the last pass; i and i + NBL/2 are partners j, H - j
    const int j = lt + TPF * (i % (NBL / 2));
    return i < NBL / 2 ? j : (j == 0 ? H / 2 : H - j);
  };
  const bool special = lt == 0;  // butterflies 0 and H/2: each is its own partner
  auto k_split = [&](int i, int q) {
    return special && i == 0 && q >= RL / 2 ? H / 2 + H * (q - RL / 2) : lt + TPF * i + H * q;
  };
  float2 tm[R2];
  if constexpr (R3 > 1) {
#pragma unroll
    for (int r = 1; r < R2; ++r) tm[r] = tw[(lt % R1) * r * (2 * M / (R1 * R2))];
  }

  f32x2_u z[V];  // samples of the frame that comes next
  auto load_next = [&](int advance) {  // `advance`: frames to the one after it
    const bool past = b >= P.g.B;  // behind the last frame: that frame again, never written
    const int i0 = (past ? T - 1 : t) * P.g.hop - P.g.pad;
    const float* __restrict__ xb = P.g.x + (past ? P.g.B - 1 : b) * P.g.L;
    // Pairs as vectors: as two floats each, the compiler joined both ways of this branch to 32 words requested one by one at 32 addresses
    // computed ahead (1,770 x 176,400 samples 1.51 -> 1.35 ms, N = 1,024 complex 300 x 176,400 428 -> 369 us, N = 4,096 Mel 1.72 -> 1.58 ms).
    if (__builtin_amdgcn_ballot_w64(i0 < 0 || i0 + 2 * M > L) == 0) {
#pragma unroll
      for (int i = 0; i < V; ++i) z[i] = *reinterpret_cast<const f32x2_u*>(xb + i0 + 2 * (lt + TPF * (i / R1) + (M / R1) * (i % R1)));
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const int m = i0 + 2 * (lt + TPF * (i / R1) + (M / R1) * (i % R1));
        z[i] = (f32x2_u){xb[reflect(m, L)], xb[reflect(m + 1, L)]};
      }
      if constexpr (WAIT) __builtin_amdgcn_s_waitcnt(0x0f70);
    }
    t += advance;
    if (t >= T) {
      const int q = t - T < T ? 1 : t / T;
      t -= q * T;
      b += q;
    }
  };
  const int to_next = ((stride - 1) << P.lg_tf) + FPWG;  // from a tile's last step to the next tile's first
  load_next(iters > 1 ? FPWG : to_next);
  // The tile before this one is written out (or taken to Mel bands) a part after every step, while the stores of the parts
  // before are on their way: a step of its own for it, between two barriers, had all the chip's workgroups computing and then
  // all of them storing (1,770 x 176,400 samples: 2.20 ms).
  long long pb0 = 0, p_left = 0;
  int pt0 = 0;
  // Waves whose frames are their own wait for each other through two counters, of the waves' tiles computed and of their tiles
  // written out, and only for what they are about to touch: a wave may be a step ahead of another.  Meeting at a barrier once a
  // tile keeps them all in the same pass, on the same pipe (1,770 x 176,400 samples, without any output: 1.22 ms against 0.82).
  int* const computed = reinterpret_cast<int*>(tile + P.sync_word);
  int* const written = computed + 1;
  if (tid < 2) computed[tid] = 0;
  __syncthreads();
  auto signal = [&](int* counter) {
    wave_fence();
    if (lane == 0) __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto wait = [&](const int* counter, int until) {
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < until) __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    __builtin_amdgcn_wave_barrier();
  };
  constexpr bool FLAGS = TPF <= 64;
  // written out in the first steps of the next tile, so that no wave waits for another's last one
  const int lg_parts = iters > 1 && !P.at_once ? 30 - __builtin_clz(iters) : 0, parts = 1 << lg_parts;
  auto emit = [&](const float* done, int part) {
    if constexpr (MODE == FFT_MODE_MEL) {
      if (P.mel_lds)
        mel_tile(P, mel, melw, done, C::PITCH, P.lg_tf, p_left, pb0, pt0, wave, n_wave, lane, part, lg_parts);
      else
        mel_tile(P, P.mel, P.melw, done, C::PITCH, P.lg_tf, p_left, pb0, pt0, wave, n_wave, lane, part, lg_parts);
      if (P.spec)
        store_tile<FFT_MODE_MEL>(done, C::PITCH, 0, P.lg_tf, M + 1, P.spec, NNA_OUT_POWER, p_left, pb0, pt0, T, wave, n_wave, lane, part, lg_parts);
    } else {
      const int rows = MODE == FFT_MODE_CPLX && P.fmt == NNA_OUT_COMPLEX ? 2 * (M + 1) : M + 1;
      store_tile<MODE>(done, C::PITCH, C::PLANE, P.lg_tf, rows, P.out, P.fmt, p_left, pb0, pt0, T, wave, n_wave, lane, part, lg_parts);
    }
  };
  [[maybe_unused]] int step = 0;
  int n_done = 0;  // n_wave times the tiles this wave has computed

  // What is in flight here counts as in flight at the head of every step, where the compiler then waits for all requests, and with them for
  // the stores of the step before.  Waited for once, before the loop: 1 x 3,969,031 samples, N = 1,024, complex, 31.0 -> 29.6 us; Mel 64 x
  // 110,250, N = 2,048, 38.4 -> 37.0; 1,770 x 80,000, N = 4,096, 512 bands, 1.59 -> 1.52 ms; magnitudes, N = 256, 500 x 176,400, 436 -> 397 us.
  // Longer rows are the exception: waves that run ahead of their stores spread the halves of a line over more time, and rows that begin anywhere
  // in a line take 1.51 ms for 1.35 (N = 2,048, 1,770 x 345 frames) and 1.27 for 0.91 (N = 4,096, 500 x 345).  (Rows of whole lines gain: of 352 frames
  // 1.19 for 1.33.  They run as the others of their window.)
  if constexpr (MODE == FFT_MODE_MEL || M < 1024) __builtin_amdgcn_s_waitcnt(0x0f70);
  float *cur = tile, *old = tile + P.buf_words;
  for (long long tile_i = lo; tile_i < hi; tile_i += stride) {
    if (FLAGS && n_done > n_wave) wait(written, n_done - n_wave);  // the buffer's last tile
    for (int it = 0; it < iters; ++it) {
      // The two waves of a SIMD take the lead in turn.  Left to themselves the older one always has it, and waits for the other at
      // the end of its tile (1,770 x 176,400 samples: 1.63 -> 1.50 ms).
      if constexpr (C::WAVES == 8 || TPF > 64) {
        if ((wave >> 2 ^ step++) & 1)
          __builtin_amdgcn_s_setprio(1);
        else
          __builtin_amdgcn_s_setprio(0);
      }
      float* __restrict__ reg = cur + (it * FPWG + first) * C::PITCH;
      cplx a[V];
#pragma unroll
      for (int i = 0; i < V; ++i) a[i] = {z[i].x * w[i].x, z[i].y * w[i].y};
      load_next(it + 2 == iters || iters == 1 ? to_next : FPWG);
      __builtin_amdgcn_sched_barrier(0);  // (the requests stay in front of the passes: 1.67 -> 1.51 ms)
      // pass 1
#pragma unroll
      for (int p = 0; p < V / R1; ++p) {
        cplx v[R1];
#pragma unroll
        for (int r = 0; r < R1; ++r) v[r] = a[p * R1 + r];
        dft<R1>(v);
#pragma unroll
        for (int r = 0; r < R1; ++r) a[p * R1 + r] = v[r];
      }
      // values of one pass go to words out(i) and come back from in(i)
      auto exchange = [&](auto out, auto in) {
        fence();
#pragma unroll
        for (int i = 0; i < V; ++i) reg[out(i)] = a[i].x;
        fence();
        float re[V];
#pragma unroll
        for (int i = 0; i < V; ++i) re[i] = reg[in(i)];
        fence();
#pragma unroll
        for (int i = 0; i < V; ++i) reg[out(i)] = a[i].y;
        fence();
#pragma unroll
        for (int i = 0; i < V; ++i) a[i] = {re[i], reg[in(i)]};
        wave_fence();
      };
      // value v sits in word padded(v) = v + v / 16: the strides R1 of the first pass's results do not collide on the banks.
      // Written as a base per butterfly and constant steps:
      auto out1 = [&](int i) { return padded((lt + TPF * (i / R1)) * R1) + i % R1; };       // j R1 + r, r < R1 <= 16
      auto in_last = [&](int i) { return padded(j_last(i / RL)) + padded(H * (i % RL)); };  // H a multiple of 16, or j < H = 8
      if constexpr (R3 > 1) {
        exchange(out1, [&](int i) { return padded(lt + TPF * (i / R2)) + padded((M / R2) * (i % R2)); });
#pragma unroll
        for (int p = 0; p < V / R2; ++p) {
          cplx v[R2];
          v[0] = a[p * R2];
#pragma unroll
          for (int r = 1; r < R2; ++r) v[r] = twiddle(a[p * R2 + r], tm[r]);
          dft<R2>(v);
#pragma unroll
          for (int r = 0; r < R2; ++r) a[p * R2 + r] = v[r];
        }
        exchange(
            [&](int i) {
              const int j = lt + TPF * (i / R2);
              return padded((j / R1) * (R1 * R2)) + j % R1 + padded((i % R2) * R1);  // j % R1 < R1, R1 = 8 or 16
            },
            in_last);
      } else {
        exchange(out1, in_last);
      }
      // last pass
#pragma unroll
      for (int p = 0; p < NBL; ++p) {
        cplx v[RL];
        v[0] = a[p * RL];
#pragma unroll
        for (int r = 1; r < RL; ++r) v[r] = twiddle(a[p * RL + r], tl[p * (RL - 1) + r - 1]);
        dft<RL>(v);
#pragma unroll
        for (int r = 0; r < RL; ++r) a[p * RL + r] = v[r];
      }
      fence();
      // bins k and M - k
      auto put = [&](int k, cplx x) {
        if constexpr (MODE == FFT_MODE_CPLX) {
          reg[k] = x.x;
          reg[C::PLANE + k] = x.y;
        } else {
          float v = __builtin_fmaf(x.x, x.x, x.y * x.y);
          if constexpr (MODE == FFT_MODE_MEL) {
            if (P.mel_power == 1) v = __builtin_amdgcn_sqrtf(v);
          }
          reg[k] = v;
        }
      };
#pragma unroll
      for (int i = 0; i < NBL / 2; ++i) {
        const cplx* A = a + i * RL;
        const cplx* B = a + (i + NBL / 2) * RL;
#pragma unroll
        for (int q = 0; q < RL; ++q) {
          cplx zk = A[q], zm = B[RL - 1 - q];
          if (i == 0) {  // lane 0 of a frame: the pairs inside butterfly 0, then those inside butterfly H/2
            const cplx sk = q < RL / 2 ? A[q] : B[q - RL / 2];
            const cplx sm = q < RL / 2 ? A[(RL - q) % RL] : B[RL - 1 - (q - RL / 2)];
            zk = {special ? sk.x : zk.x, special ? sk.y : zk.y};
            zm = {special ? sm.x : zm.x, special ? sm.y : zm.y};
          }
          cplx xk, xm;
          const int k = k_split(i, q);
          split_pair(zk, zm, ts[i * RL + q], xk, xm);
          put(k, xk);
          put(M - k, xm);
        }
      }
      if (special) put(M / 2, cplx{2.f * a[RL / 2].x, -2.f * a[RL / 2].y});
      if constexpr (MODE == FFT_MODE_MEL) {
        if (lt < 3) reg[M + 1 + lt] = 0.f;  // bins a band's last quad of weights may pad into
      }
      // the next frame's samples, requested at the start of this step, are waited for here: behind the stores below the wait would
      // be for those too
#pragma unroll
      for (int i = 0; i < V; ++i) asm volatile("" : "+v"(z[i]));
      if (p_left > 0 && it < parts) {
        if (FLAGS && it == 0) wait(computed, n_done);
        emit(old, it);
        if (FLAGS && it == parts - 1) signal(written);
      }
    }
    n_done += n_wave;
    if (FLAGS)
      signal(computed);
    else
      __syncthreads();  // this tile is complete, and the one before it written out
    pb0 = b0;
    pt0 = t0;
    p_left = P.g.n_frames - (tile_i << P.lg_tf);
    if (!FLAGS && P.at_once) {
      emit(cur, 0);
      __syncthreads();
      p_left = 0;
    }
    float* const swap = cur;
    cur = old;
    old = swap;
    frame_of(stride << P.lg_tf, b0, t0, T, b0, t0);
  }
  if (FLAGS) wait(computed, n_done);
  for (int it = 0; it < parts; ++it) emit(old, it);
}

// ---------------------------------------------------------------------------------------
// Any other N = 2 M whose M has no prime factor above 7 and fits in LDS: one wave per frame, radices from a list,
// every pass from one LDS buffer to the other.  200 x 176,400 samples against the contraction it replaces: N = 400, hop 160
// 802 -> 435 us; N = 1,000, hop 250 2.5 ms -> 781 us; N = 8,192, hop 2,048 5.3 -> 3.5 ms.
// ---------------------------------------------------------------------------------------
template <int R>
__device__ __forceinline__ void general_pass(const cplx* __restrict__ src, cplx* __restrict__ dst, int M, int Ns, float inv_ns,
                                             const float2* __restrict__ tw, int lane) {
  const int nb = M / R, stride = 2 * M / (Ns * R);
  for (int j = lane; j < nb; j += 64) {
    const int jq = (int)((j + 0.5f) * inv_ns), jr = j - jq * Ns;
    cplx v[R];
    v[0] = src[j];
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = twiddle(src[j + nb * r], tw[jr * r * stride]);
    dft<R>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) dst[jq * Ns * R + jr + r * Ns] = v[r];
  }
}

template <int MODE>
__global__ __launch_bounds__(256, 2) void fft_general_kernel(FftParams P) {
  extern __shared__ float lds[];
  const int M = P.M, L = (int)P.g.L, T = P.g.T, pitch = P.pitch;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int TF = 1 << P.lg_tf;
  float* tile = lds;
  cplx* buf0 = reinterpret_cast<cplx*>(lds + ((TF * pitch + 1) & ~1)) + (size_t)wave * 2 * M;
  cplx* buf1 = buf0 + M;
  const long long lo = P.n_tiles * blockIdx.x / gridDim.x, hi = P.n_tiles * (blockIdx.x + 1) / gridDim.x;
  const float2* __restrict__ win = reinterpret_cast<const float2*>(P.win);
  for (long long tile_i = lo; tile_i < hi; ++tile_i) {
    const long long f0 = tile_i << P.lg_tf;
    const long long b0 = (unsigned long long)f0 / (unsigned)T;
    const int t0 = (int)(f0 - b0 * T);
    for (int fi = wave; fi < TF && f0 + fi < P.g.n_frames; fi += nw) {
      long long b;
      int t;
      frame_of(fi, b0, t0, T, b, t);
      const int i0 = t * P.g.hop - P.g.pad;
      const float* __restrict__ xb = P.g.x + b * P.g.L;
      wave_fence();
      if (i0 >= 0 && i0 + 2 * M <= L) {
        for (int m = lane; m < M; m += 64) {
          cplx v;
          __builtin_memcpy(&v, xb + i0 + 2 * m, 8);
          buf0[m] = {v.x * win[m].x, v.y * win[m].y};
        }
      } else {
        for (int m = lane; m < M; m += 64)
          buf0[m] = {xb[reflect(i0 + 2 * m, L)] * win[m].x, xb[reflect(i0 + 2 * m + 1, L)] * win[m].y};
      }
      cplx *src = buf0, *dst = buf1;
      int Ns = 1;
      for (int p = 0; p < P.n_radix; ++p) {
        wave_fence();
        const int R = P.radix[p];
        const float inv = 1.0f / (float)Ns;
        if (R == 8) general_pass<8>(src, dst, M, Ns, inv, P.tw, lane);
        else if (R == 4) general_pass<4>(src, dst, M, Ns, inv, P.tw, lane);
        else if (R == 5) general_pass<5>(src, dst, M, Ns, inv, P.tw, lane);
        else if (R == 3) general_pass<3>(src, dst, M, Ns, inv, P.tw, lane);
        else if (R == 7) general_pass<7>(src, dst, M, Ns, inv, P.tw, lane);
        else general_pass<2>(src, dst, M, Ns, inv, P.tw, lane);
        Ns *= R;
        cplx* s = src;
        src = dst;
        dst = s;
      }
      wave_fence();
      float* __restrict__ row = tile + fi * pitch;
      auto put = [&](int k, cplx x) {
        if constexpr (MODE == FFT_MODE_CPLX) {
          row[k] = x.x;
          row[M + 1 + k] = x.y;
        } else {
          const float v = __builtin_fmaf(x.x, x.x, x.y * x.y);
          row[k] = MODE == FFT_MODE_MEL && P.mel_power == 1 ? __builtin_amdgcn_sqrtf(v) : v;
        }
      };
      for (int k = lane; k <= M / 2; k += 64) {
        cplx xk, xm;
        split_pair(src[k], src[k == 0 ? 0 : M - k], P.tw[k], xk, xm);
        put(k, xk);
        put(M - k, xm);
      }
      if constexpr (MODE == FFT_MODE_MEL) {
        if (lane < 3) row[M + 1 + lane] = 0.f;
      }
    }
    __syncthreads();
    if constexpr (MODE == FFT_MODE_MEL) {
      mel_tile(P, P.mel, P.melw, tile, pitch, P.lg_tf, P.g.n_frames - f0, b0, t0, wave, nw, lane, 0, 0);
      if (P.spec)
        store_tile<FFT_MODE_MEL>(tile, pitch, 0, P.lg_tf, M + 1, P.spec, NNA_OUT_POWER, P.g.n_frames - f0, b0, t0, T, wave, nw, lane, 0, 0);
    } else {
      const int rows = MODE == FFT_MODE_CPLX && P.fmt == NNA_OUT_COMPLEX ? 2 * (M + 1) : M + 1;
      store_tile<MODE>(tile, pitch, M + 1, P.lg_tf, rows, P.out, P.fmt, P.g.n_frames - f0, b0, t0, T, wave, nw, lane, 0, 0);
    }
    __syncthreads();
  }
}

// Grid and tile of a launch: the steps per tile are halved until there are 512 tiles, two per CU, or one step is left; small
// tiles spread a short batch over the chip, large ones write longer runs.
void shape_launch(FftParams& P, int frames_per_step, int max_iters) {
  int iters = max_iters;
  while (iters > 1 && P.g.n_frames < 512LL * frames_per_step * iters) iters >>= 1;
  int tf = frames_per_step * iters, lg = 0;
  while ((1 << lg) < tf) ++lg;
  P.lg_tf = lg;
  P.n_tiles = (P.g.n_frames + tf - 1) / tf;
}

// Samples of frames that reach past a waveform's ends, left in flight, are what the compiler waits for ahead of the other frames' requests, and with
// them for every store before: where one frame in twenty or fewer is one, they are waited for at once instead (300 x 176,400 samples, N = 512, hop 128,
// magnitudes 213 -> 202 us; N = 128 to 4,096 0.97 .. 1.02 of the time).  Where they are the rule, that is a wait in every step: 1,116 x 990, N = 256, Mel,
// 19.5 -> 22.2 us, 50,855 x 335, N = 512, phases 304 -> 332; of one frame in ten 0.95 .. 1.0 of the time without, of all 0.86 .. 1.0.
bool few_ends(const FftParams& P) {
  const long long N = 2LL * P.M, hop = P.g.hop, pad = P.g.pad, first = (pad + hop - 1) / hop;  // first frame inside, and the first past the last one
  const long long behind = P.g.L + pad >= N ? std::min<long long>(P.g.T, (P.g.L + pad - N) / hop + 1) : 0;
  return 20 * (P.g.T - std::max(0LL, behind - first)) <= P.g.T;
}

template <typename S, int MODE>
hipError_t launch_fixed(FftParams& P, hipStream_t stream) {
  using C = typename S::template Tile<MODE>;
  // a batch too short for every CU to take a step spreads over twice as many in workgroups of half the size
  const int n_wave = P.g.n_frames > 256LL * C::frames_per_step(4) ? C::WAVES : 4, step = C::frames_per_step(n_wave);
  const int groups = C::WAVES == 8 ? 256 : 512;
  // Largest tile whose workgroups are done about as early as with smaller ones
  auto longest = [&](int steps) { return (P.g.n_frames + (long long)groups * steps * step - 1) / ((long long)groups * steps * step) * steps; };
  const int tables = MODE == FFT_MODE_MEL ? (P.n_mels + P.mel_quads) * 16 : 0;
  P.mel_lds = tables > 0 && 2 * step * C::PITCH * 4 + 32 + tables <= C::LDS;
  int iters = C::max_steps(n_wave, 32 + (P.mel_lds ? tables : 0));
  // Frames of two waves (N = 4,096) whose LDS holds two buffers of one step, two frames, only: one buffer of two steps, where a workgroup
  // takes several tiles.  Rows of four frames are written in half the requests and the bands' lanes are filled: 140,000 frames, complex,
  // 2.83 ms (four frames, stored between two barriers) -> 3.14 (two buffers) -> 2.41; Mel, 40 bands 1.00 -> 1.45 -> 1.02, 128: 0.90 -> 1.00
  // -> 0.77, 512: 1.06 -> 0.93 -> 0.90.  Several: of two steps for bands and phases, which are computed on the way out (1,384 frames: 23.4
  // us -> 27.0, 80 bands 21.0 -> 25.1), of one for complex rows (30.6 -> 28.4).  Four steps leave the Mel tables in memory (1.07 to 1.1
  // times the time), for bands that fill the lanes better by more than that: 80 bands 0.92 -> 1.12 -> 1.00 ms in two steps, 0.91 in four.
  const bool computed_out = MODE == FFT_MODE_MEL || (MODE == FFT_MODE_CPLX && P.fmt == NNA_OUT_PHASE);
  if (C::TPF > 64 && iters == 1 && P.g.n_frames > (long long)groups * step * (computed_out ? 2 : 1)) {
    auto rounds = [&](int steps) { return (P.n_mels * step * steps + 64 * n_wave - 1) / (64 * n_wave); };  // of a tile's bands
    P.at_once = 1;
    iters = MODE == FFT_MODE_MEL && 4 * step * C::PITCH * 4 + 16 <= C::LDS && 11 * rounds(4) < 20 * rounds(2) ? 4 : 2;
  }
  // Twice the steps where the longest workgroup takes no more than these times what it would take without.  Two steps for one: at 4 / 3
  // between 9 % more and 20 % less time (n_fft 512 to 4,096, 6,000 to 20,000 frames), at twice as many 20 to 45 % more; from one buffer at
  // 1.2 11 % less time for 40 bands and 10 % more for 512, at 1.11 between 19 % less and 2 % more.  Four for two, 80 bands: at 1.01 9 % less,
  // at 1.11 1 %, at 1.2 4 % more.
  auto limit = [&] { return iters == 2 ? (P.at_once && computed_out ? 1.15 : 1.4) : P.at_once ? 1.1 : 1.0; };
  while (iters > 1 && (longest(iters) > limit() * longest(iters / 2) || (P.at_once && iters == 4 && longest(4) > 1.15 * longest(1)))) iters >>= 1;
  if (iters == 1) P.at_once = 0;
  if (P.at_once && iters == 4) P.mel_lds = 0;
  const int tf = step * iters;
  P.lg_tf = 0;
  while ((1 << P.lg_tf) < tf) ++P.lg_tf;
  P.n_tiles = (P.g.n_frames + tf - 1) / tf;
  const long long grid = std::min<long long>((P.n_tiles + 7) / 8 * 8, groups);
  const int words = (tf * C::PITCH + 3) & ~3;
  P.buf_words = P.n_tiles > grid && !P.at_once ? words : 0;
  P.sync_word = words + P.buf_words;
  if (P.mel_lds) P.mel_lds = P.sync_word + 4;
  const size_t bytes = (size_t)(P.sync_word + 4) * 4 + (P.mel_lds ? tables : 0);
  clear_stale_error();
  if (few_ends(P))
    hipLaunchKernelGGL((fft_kernel<S::M, S::R1, S::R2, S::R3, S::V, MODE, true>), dim3((unsigned)grid), dim3(64 * n_wave), bytes, stream, P);
  else
    hipLaunchKernelGGL((fft_kernel<S::M, S::R1, S::R2, S::R3, S::V, MODE, false>), dim3((unsigned)grid), dim3(64 * n_wave), bytes, stream, P);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(FftParams& P, hipStream_t stream) {
  hipError_t e = hipSuccess;
  if (with_shape(P.M, [&](auto s) { e = launch_fixed<decltype(s), MODE>(P, stream); })) return e;
  const size_t row = (size_t)P.pitch * 4, work = (size_t)P.M * 16;
  int nw = 4, tf = 16;
  while (nw > 1 && nw * work + nw * row > (size_t)kLdsTwo) nw >>= 1;
  while (tf > nw && nw * work + tf * row > (size_t)kLdsTwo) tf >>= 1;
  shape_launch(P, nw, std::max(1, tf / nw));
  const size_t bytes = nw * work + ((((size_t)P.pitch << P.lg_tf) + 1) & ~(size_t)1) * 4;
  clear_stale_error();
  hipLaunchKernelGGL((fft_general_kernel<MODE>), dim3((unsigned)std::min<long long>(P.n_tiles, 1024)), dim3(64 * nw), bytes, stream, P);
  return hipGetLastError();
}

// every launch that may ask for more than 64 KB has leave to
template <int MODE>
hipError_t allow_lds_mode() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fft_general_kernel<MODE>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
  for (const int M : kShapes)
    with_shape(M, [&](auto s) {
      using S = decltype(s);
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(fft_kernel<S::M, S::R1, S::R2, S::R3, S::V, MODE, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsAll);
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(fft_kernel<S::M, S::R1, S::R2, S::R3, S::V, MODE, false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsAll);
    });
  return e;
}

}  // namespace

// The order in which the lanes of a frame take their twiddles in fft_kernel<M>: those of the last pass, then of the bins.
template <typename S>
void lane_twiddles(std::vector<int>& index) {
  using C = typename S::template Tile<FFT_MODE_POWER>;
  constexpr int V = S::V, RL = C::RL, H = C::H, TPF = C::TPF, NBL = C::NBL;
  static_assert(NBL * (RL - 1) % 2 == 0 && V % 4 == 0, "twiddles in pairs");
  index.resize((size_t)TPF * (NBL * (RL - 1) + V / 2));
  for (int lt = 0; lt < TPF; ++lt) {
    int u = 0;
    auto add = [&](int k) {
      index[((size_t)(u / 2) * TPF + lt) * 2 + u % 2] = k;
      ++u;
    };
    for (int p = 0; p < NBL; ++p) {
      const int jA = lt + TPF * (p % (NBL / 2)), j = p < NBL / 2 ? jA : (jA == 0 ? H / 2 : H - jA);
      for (int r = 1; r < RL; ++r) add(2 * j * r);
    }
    for (int i = 0; i < NBL / 2; ++i)
      for (int q = 0; q < RL; ++q) add(lt == 0 && i == 0 && q >= RL / 2 ? H / 2 + H * (q - RL / 2) : lt + TPF * i + H * q);
  }
}

void fft_lane_twiddles(int M, std::vector<int>& index) {
  index.clear();
  with_shape(M, [&](auto s) { lane_twiddles<decltype(s)>(index); });
}

bool fft_radices(int n_fft, int (&radix)[16], int& n_radix) {
  // Below 64 samples a wave per frame is mostly idle: N = 32, hop 32 took 374 us where the contraction takes 77 (100 x 176,400)
  if (n_fft < 64 || (n_fft & 1)) return false;
  int m = n_fft / 2;
  if ((size_t)m * 16 + (size_t)(2 * m + 8) * 4 > (size_t)kLdsMax) return false;
  n_radix = 0;
  for (const int r : {8, 7, 5, 4, 3, 2})
    while (m % r == 0) {
      radix[n_radix++] = r;
      m /= r;
    }
  return m == 1;
}

hipError_t launch_stft_fft(FftParams& P, int mode, hipStream_t stream) {
  const int words = mode == FFT_MODE_CPLX ? 2 * P.M + 2 : P.M + 4;
  P.pitch = words | 1;
  switch (mode) {
    case FFT_MODE_POWER: return launch_mode<FFT_MODE_POWER>(P, stream);
    case FFT_MODE_CPLX: return launch_mode<FFT_MODE_CPLX>(P, stream);
    default: return launch_mode<FFT_MODE_MEL>(P, stream);
  }
}

hipError_t fft_kernels_init() {
  hipError_t e = allow_lds_mode<FFT_MODE_POWER>();
  if (e == hipSuccess) e = allow_lds_mode<FFT_MODE_CPLX>();
  if (e == hipSuccess) e = allow_lds_mode<FFT_MODE_MEL>();
  return e;
}

}  // namespace nna
