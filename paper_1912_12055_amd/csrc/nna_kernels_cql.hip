// Constant-Q transform with time-domain kernels (Sec. III-C, eq. (CQT)), the kernels as combinations of a few functions per hop.
//
// A kernel of N_k taps spans J hops, and cut at the hops' boundaries the kernels of 16 neighbouring bins are J x 32 rows of `hop`
// taps.  Far fewer dimensions hold them all, as closely as float32 taps would (nna_banks.hip), because within one hop a low bin's
// kernel is a smooth function.  With U an orthonormal basis of that space and A the coordinates,
//     y[b][i] = sum_c U[i][c] x[b hop + c]          i < r, every hop-block b of the padded waveform
//     C_k[t]  = sum_j sum_i A_k[j][i] y[t + j][i].
// 168 bins of 24 per octave at 44.1 kHz, hop 512: 0.7 million multiply-adds per frame against 1.6 million of the kernels folded about
// their centres (nna_kernels_cqf.hip) and 3.2 million of the kernels as they stand.
//
// Short kernels, where the first stage alone would cost more than their taps, stay as they are: direct items of up to 32 bins.
//
// A workgroup takes one item (16 bins) and one tile of 64 FB frames.  Stage 1 (basis rows x hop-blocks) reads its hop-blocks from
// the waveform straight into registers in operand order -- sixteen hops per load, 64 bytes of each -- and writes y to LDS, a hop's r
// coordinates in a row.  Stage 2 then is the convolution of the direct kernel with a hop of r samples: the taps of a frame are r J
// consecutive words of LDS, so r needs no padding to the taps of a step, only to 4 modulo 8, which keeps the rows of sixteen frames on
// different banks.
//
// Both run on v_mfma_f32_16x16x32_bf16, every float32 as three bfloat16 (exact from 2^-110 up to 3.396e38; below, low bits are lost, above
// the first part is infinite and the sum is taken again in float32) and the six products that matter of nine: 32 taps in 96 cycles of a
// SIMD's pipe against 256 as eight v_mfma_f32_16x16x4_f32.  The weights are split with the plan, the samples on the way into the
// instruction.  Coordinates are split once, on the way into LDS, by the items that need six bytes for each in no more LDS than the
// launch's largest item takes at four: small bases; the others' are split by every frame that reads them (two of the six items with a
// basis of the first and the last call below).
//
// Every sum is taken in blocks of 32 products (six instructions), each from zero and then added to a total: a chain of a thousand
// roundings was off by up to 9e-7 of a bin's norm, more than the folded kernel's half as many in the bins taken tap by tap; the
// blocks are off by 3e-7 at most.  Against 64 bits the bfloat16 form's errors are 0.5 .. 0.9 of the float32 instruction's, eight
// configurations, six signals each.
//
// Bound by no one pipe at the batch below: the samples' splits keep the vector ALUs 52 % busy, the matrix pipe is at 39 %; a short batch
// by latency, a workgroup or two per CU.  1,770 x 176,400 samples, 168 bins of 24 per octave (MI355X): 24.5 ms
// folded about the centres, 8.25 here in float32, 6.59 in bfloat16 with every coordinate split by each frame that reads it, now 5.74;
// 16 x 220,500, 84 bins of 12 per octave: 300 -> 67.8 -> 53.8 us; the dense composed kernels of the frequency-domain layer (16 x
// 220,500, 16,384 taps): 566 -> 183 -> 138 us.  With the short kernels by tiles of nna_short.h (the direct items read four row blocks' weights for
// every 16 frames, and the loads' issue bound them): 5.81 -> 5.12 ms, 58 -> 46 us.
#include <type_traits>

#include "nna_short.h"

namespace nna {
namespace {

using std::integral_constant;
using True = integral_constant<bool, true>;
using False = integral_constant<bool, false>;

// lane (q, n), registers 0 .. 3 of row block b: (Re, Im) of bins 8 b + 2 q and + 1, frame n of the wave's frame block.  Returns the
// bins that are not finite, bit 2 (RB fb + rb) + u.
template <int FB, int RB>
__device__ __forceinline__ unsigned store_bins(const CqlParams& P, const CqlItem& item, const f32x4 (&acc)[FB][RB], const bool (&valid)[FB],
                                               long long f0, int wave, int q, int n) {
  const FrameGeom& g = P.g;
  unsigned odd = 0;
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) {
    if (!valid[fb]) continue;
    const long long f = f0 + wave * (16 * FB) + fb * 16 + n, b = f / g.T;
    float* __restrict__ op = P.out + b * P.out_wave_stride + (f - b * g.T);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = 8 * rb + 2 * q + u;
        if (k >= item.n_bins) continue;
        const float re = acc[fb][rb][2 * u], im = acc[fb][rb][2 * u + 1];
        store_bin(P.fmt, P.g.T, op, item.bin0 + k, re, im);
        odd |= (finite(re) && finite(im) ? 0u : 1u) << (2 * (RB * fb + rb) + u);
      }
  }
  return odd;
}

// Short kernels, tap by tap.
template <int FB>
__device__ __forceinline__ void direct_item(const CqlParams& P, const CqlPart& part, const CqlItem& item, long long ft, float* Y) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int q = lane >> 4, n = lane & 15;
  const FrameGeom& g = P.g;
  const long long f0 = ft * part.tile_frames;
  const int m_valid = (int)((g.n_frames - f0) < part.tile_frames ? (g.n_frames - f0) : part.tile_frames);
  TileMap tm;
  tm.T = g.T;
  tm.b0 = f0 / g.T;
  tm.t0 = (int)(f0 - tm.b0 * g.T);
  tm.n0 = (g.T - tm.t0) < m_valid ? (g.T - tm.t0) : m_valid;
  tm.extra = item.jspan - 1;
  const int rows_used = tm.frame_row(m_valid - 1) + tm.extra + 1;
  const int hop = g.hop;
  constexpr int RB = 4;  // row blocks
  // this wave's frames
  bool valid[FB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) valid[fb] = wave * (16 * FB) + fb * 16 + n < m_valid;
  f32x4 acc[FB][RB];
  auto clear = [&] {
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
      for (int b = 0; b < RB; ++b) acc[fb][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  };
    // KC columns of the tile's hops at a time in LDS (row t + j serves frame t at hop-block j, as in the direct kernel), two
  // buffers; per chunk the steps of 16 taps that hold taps, each of them for the first `a` row blocks (the kernels shrink from
  // row block to row block).  The code is kept short: a workgroup runs most of it a few times only, and instructions that miss
  // their cache cost more than the work (unrolled over four chunk switches, 16 x 220,500 samples took 89 us instead of 67).
  constexpr int KC = CQL_COLS(FB), NP = CQL_PASSES(FB), PITCH = KC + 4, V = KC / 4, RPP = 256 / V;
  const int L = (int)g.L;
  const int rows_buf = (rows_used + 31) & ~31;
  const int* __restrict__ chunk0 = P.steps + item.step0;       // first step of every 32 columns, [hop / 32 + 1], multiples of four
  const int* __restrict__ steps = chunk0 + hop / 32 + 1;       // a | 16-column block << 3 | hop-block << 12
  const uint4* __restrict__ up = P.ub + item.u0 / 2 * 3 + lane;  // [pair of steps][4 row blocks][3 planes][64 lanes]
  const int cv = tid % V, r0 = tid / V;
  const float* xb[NP];  // this thread's rows: their waveform, the first of its four samples in column 0
  int pos[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int row = p * RPP + r0;
    long long b;
    int sigma;
    tm.decode(row < rows_used ? row : rows_used - 1, b, sigma);
    xb[p] = g.x + b * g.L;
    pos[p] = (sigma + item.j0) * hop - g.pad + 4 * cv;
  }
  // four samples on one side of either end are a stored run, read backwards behind an end; a run that straddles an end (only when
  // L, the hop or the padding are not multiples of 4) is read again, sample by sample, when the tile is written
  f32x4 R[NP];
  unsigned rev = 0;
  bool gen = false;
  auto request = [&](int c) {
    rev = 0;
    gen = false;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int s = pos[p] + c;
      const int src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
      rev |= (src != s ? 1u : 0u) << p;
      gen |= (unsigned)src > (unsigned)(L - 4);
      R[p] = *reinterpret_cast<const f32x4_u*>(xb[p] + (src < 0 ? 0 : src > L - 4 ? L - 4 : src));
    }
  };
  auto store = [&](int c, float* dst) {
    dst += r0 * PITCH + 4 * cv;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const f32x4 v = R[p];
      const bool r = (rev >> p) & 1u;
      if (p * RPP + r0 < rows_buf)
        *reinterpret_cast<f32x4*>(dst + p * RPP * PITCH) = (f32x4){r ? v.w : v.x, r ? v.z : v.y, r ? v.y : v.z, r ? v.x : v.w};
    }
    if (__builtin_amdgcn_ballot_w64(gen) == 0) return;
#pragma unroll 1
    for (int row = r0; row < rows_used; row += RPP) {
      long long b;
      int sigma;
      tm.decode(row, b, sigma);
      const float* __restrict__ x = g.x + b * g.L;
      const int s = (sigma + item.j0) * hop - g.pad + 4 * cv + c;
      const int src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
      if ((unsigned)src > (unsigned)(L - 4))
        for (int e = 0; e < 4; ++e) dst[(row - r0) * PITCH + e] = x[reflect_clamped(s + e, L)];
    }
  };
  int f_off[FB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) f_off[fb] = (valid[fb] ? tm.frame_row(wave * (16 * FB) + fb * 16 + n) : 0) * PITCH + 4 * q;
  // A step: 32 columns of one hop-block, for the first `a` row blocks
  auto multiply = [&](int a, const u32x4 (&w)[4][3], const f32x4 (&x)[FB][2]) {
    if (!a) return;
    Planes b[FB];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) b[fb] = split8(x[fb]);
    // row block by row block: a kernel that has ended costs a branch
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < a) {
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) acc[fb][i] += multiply_octets(w[i], b[fb], (f32x4){0.f, 0.f, 0.f, 0.f});
      }
  };
  // The weights are requested a step ahead, across chunks, and so are the frames, from LDS, within a chunk.
  const int n_pair = item.n_step / 2;
  u32x4 w[2][4][3];
  f32x4 x[2][FB][2];
  auto fetch_w = [&](int s, u32x4 (&v)[4][3]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int l = 0; l < 3; ++l) v[i][l] = *reinterpret_cast<const u32x4*>(up + (((long long)s * 4 + i) * 3 + l) * 64);
  };
  clear();
  request(0);
  fetch_w(0, w[0]);
  for (int c = 0; c < hop; c += KC) {
    float* tile = Y + ((c / KC) & 1) * rows_buf * PITCH;
    store(c, tile);
    __syncthreads();  // also: the buffer of the chunk before last has been read by every wave
    if (c + KC < hop) request(c + KC);
    const int next = (c + KC) / 32, s1 = chunk0[next < hop / 32 ? next : hop / 32] / 2;
    auto fetch_x = [&](int d, f32x4 (&v)[FB][2]) {
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          v[fb][h] = *reinterpret_cast<const f32x4*>(tile + f_off[fb] + (d >> 12) * PITCH + ((d << 1) & (KC - 32)) + 16 * h);
    };
    int s = chunk0[c / 32] / 2;
    int4 d = s < s1 ? *reinterpret_cast<const int4*>(steps + 2 * s) : make_int4(0, 0, 0, 0);
    fetch_x(d.x, x[0]);
    for (; s < s1; s += 2) {
      const int4 dn = *reinterpret_cast<const int4*>(steps + 2 * (s + 2 < n_pair ? s + 2 : s));
      const int du[3] = {d.x, d.z, dn.x};
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        fetch_w(s + u + 1 < n_pair ? s + u + 1 : n_pair - 1, w[u ^ 1]);
        // (behind the chunk's last step: a step of the next chunk, its offsets within the tile all the same; read and dropped)
        fetch_x(du[u + 1], x[u ^ 1]);
        __builtin_amdgcn_sched_barrier(0);
        multiply(du[u] & 7, w[u], x[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
      d = dn;
    }
  }
  // A sample that is not finite, or so large that its first bfloat16 is not, makes every sum that holds its step of 32 taps NaN.  Such a
  // sum is taken again over the bin's own taps in float32: the samples that are not finite alone if there are any, else all of them.
  // (66 x 481,793 samples, 168 bins, every thousandth NaN: 16 -> 25 ms; none: 0.71 either way.)
  unsigned odd = store_bins<FB, RB>(P, item, acc, valid, f0, wave, q, n);
#pragma unroll 1
  while (odd) {
    const int bit = __builtin_ctz(odd), rb = (bit >> 1) % RB, k = 8 * rb + 2 * q + (bit & 1), fi = (wave * FB + (bit >> 1) / RB) * 16 + n;
    odd &= odd - 1;
    const long long f = f0 + fi, b = f / g.T;
    const int t = (int)(f - b * g.T);
    const int2 own = P.support[item.bin0 + k];
    const float* __restrict__ xw = g.x + b * g.L;
    const float* __restrict__ u = reinterpret_cast<const float*>(P.u + item.u0 + rb * 64 + (2 * k & 15));  // (Im: the next row)
    float re = 0.f, im = 0.f;
    bool met = false;
#pragma unroll 1
    for (int all = 0; all < 2 && !met; ++all)
#pragma unroll 1
      for (int tap0 = own.x; tap0 < own.y && !(re != re && im != im); tap0 += 8) {
        float v[8];
        bool any = all;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          v[i] = xw[reflect_clamped(t * hop - g.pad + (tap0 + i < own.y ? tap0 + i : tap0), L)];
          any = any || !finite(v[i]);
        }
        if (!any) continue;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (tap0 + i >= own.y || (!all && finite(v[i]))) continue;
          // the tap's step of 16: those of 32 columns follow each other by hop-block and half
          const int at = tap0 + i - item.j0 * hop, j = at / hop, c = at - j * hop, first = chunk0[c / 32];
          const float* w = u + ((first + 2 * (j - (steps[first] >> 12)) + ((c >> 4) & 1)) * RB * 64 + ((c >> 2) & 3) * 16) * 4 + (c & 3);
          re += w[0] * v[i];
          im += w[4] * v[i];
          met = true;
        }
      }
    store_bin(P.fmt, g.T, P.out + b * P.out_wave_stride + t, item.bin0 + k, re, im);
  }
}

// Kernels as combinations of the item's basis.
template <int FB>
__device__ __forceinline__ void lowrank_item(const CqlParams& P, const CqlPart& part, const CqlItem& item, long long ft, float* Y) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int q = lane >> 4, n = lane & 15;
  const FrameGeom& g = P.g;
  const long long f0 = ft * part.tile_frames;
  const int m_valid = (int)((g.n_frames - f0) < part.tile_frames ? (g.n_frames - f0) : part.tile_frames);
  TileMap tm;
  tm.T = g.T;
  tm.b0 = f0 / g.T;
  tm.t0 = (int)(f0 - tm.b0 * g.T);
  tm.n0 = (g.T - tm.t0) < m_valid ? (g.T - tm.t0) : m_valid;
  tm.extra = item.jspan - 1;
  const int rows_used = tm.frame_row(m_valid - 1) + tm.extra + 1;
  const int r = item.r;
  constexpr int RB = 2;  // row blocks
  // Where the launch's LDS, sized for its largest item at four bytes a coordinate, has room for six, they are kept as the three bfloat16
  // stage 2 multiplies, split once instead of once per hop-block that reads them; planes of p_words values.
  const int p_words = rows_used * r + 32;
  const bool split = 6 * p_words <= 4 * P.lds_floats;
  unsigned short* const Yb = reinterpret_cast<unsigned short*>(Y);
  const int L = (int)g.L, hop = g.hop;
  // acc[p][i] += 16 rows of weights (i) x 16 runs of samples (p) over columns [c_begin, c_end), 32 at a time.  A lane's run starts
  // at sample pos[p] of its waveform, xb[p] points there (EDGE: at the waveform; some run of the wave touches a mirrored end).
  // `u`: [chunk][u_blocks][3 planes][64 lanes], of which the first IB blocks are used.
  auto contract = [&](auto edge_tag, auto ib_tag, auto& acc, const auto& xb, const auto& pos, const uint4* u, int u_blocks,
                      int c_begin, int c_end) {
    constexpr bool EDGE = decltype(edge_tag)::value;
    constexpr int IB = decltype(ib_tag)::value, NB = sizeof(acc) / sizeof(acc[0]);
    const uint4* up = u + lane;
    auto fetch = [&](int c, f32x4 (&x)[NB][2], u32x4 (&w)[IB][3], unsigned& rev) {
      const uint4* uc = up + (long long)((c - c_begin) >> 5) * u_blocks * 192;
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int l = 0; l < 3; ++l) w[i][l] = *reinterpret_cast<const u32x4*>(uc + (3 * i + l) * 64);
      if constexpr (!EDGE) {
#pragma unroll
        for (int p = 0; p < NB; ++p) {
          x[p][0] = *reinterpret_cast<const f32x4_u*>(xb[p] + c);
          x[p][1] = *reinterpret_cast<const f32x4_u*>(xb[p] + c + 16);
        }
      } else {
        // four samples on one side of either end are a stored run, read backwards behind an end (turned round when they are used:
        // a request is not waited for here)
        rev = 0;
        bool gen = false;
#pragma unroll
        for (int p = 0; p < NB; ++p)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int s = pos[p] + c + 16 * h;
            const int src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
            rev |= (src != s ? 1u : 0u) << (2 * p + h);
            gen |= (unsigned)src > (unsigned)(L - 4);
            const int at = src < 0 ? 0 : src > L - 4 ? L - 4 : src;
            x[p][h] = *reinterpret_cast<const f32x4_u*>(xb[p] + at);
          }
        // runs that straddle an end (only when L, the hop or the padding are not multiples of 4): sample by sample
        if (__builtin_amdgcn_ballot_w64(gen) != 0) {
#pragma unroll
          for (int p = 0; p < NB; ++p)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int s = pos[p] + c + 16 * h;
              const int src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
              if ((unsigned)src > (unsigned)(L - 4)) {
                rev &= ~(1u << (2 * p + h));
#pragma unroll
                for (int e = 0; e < 4; ++e) x[p][h][e] = xb[p][reflect_clamped(s + e, L)];
              }
            }
        }
      }
    };
    auto multiply = [&](f32x4 (&x)[NB][2], const u32x4 (&w)[IB][3], unsigned rev) {
      if constexpr (EDGE) {
#pragma unroll
        for (int p = 0; p < NB; ++p)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const f32x4 v = x[p][h];
            const bool r = (rev >> (2 * p + h)) & 1u;
            x[p][h] = (f32x4){r ? v.w : v.x, r ? v.z : v.y, r ? v.y : v.z, r ? v.x : v.w};
          }
      }
#pragma unroll
      for (int p = 0; p < NB; ++p) {
        const Planes b = split8(x[p]);
#pragma unroll
        for (int i = 0; i < IB; ++i) acc[p][i] += multiply_octets(w[i], b, (f32x4){0.f, 0.f, 0.f, 0.f});
      }
    };
    if (c_begin >= c_end) return;
    // two register sets: the next 32 columns are requested ahead of this chunk's matrix instructions
    f32x4 x0[NB][2], x1[NB][2];
    u32x4 w0[IB][3], w1[IB][3];
    unsigned r0 = 0, r1 = 0;
    fetch(c_begin, x0, w0, r0);
    for (int c = c_begin; c < c_end; c += 64) {
      fetch(c + 32 < c_end ? c + 32 : c, x1, w1, r1);
      __builtin_amdgcn_sched_barrier(0);
      multiply(x0, w0, r0);
      __builtin_amdgcn_sched_barrier(0);
      if (c + 32 >= c_end) break;
      fetch(c + 64 < c_end ? c + 64 : c, x0, w0, r0);
      __builtin_amdgcn_sched_barrier(0);
      multiply(x1, w1, r1);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // this wave's frames
  bool valid[FB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) valid[fb] = wave * (16 * FB) + fb * 16 + n < m_valid;
  f32x4 acc[FB][RB];
  auto clear = [&] {
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
      for (int b = 0; b < RB; ++b) acc[fb][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  };
  // ---- stage 1: the hop-blocks' coordinates -------------------------------------------
  // NB x IB tiles of 16 hop-blocks x 16 basis functions
  auto sweep = [&](auto edge_tag, auto nb_tag, auto ib_tag, int blk0, int ib0) {
    constexpr bool EDGE = decltype(edge_tag)::value;
    constexpr int NB = decltype(nb_tag)::value, IB = decltype(ib_tag)::value;
    const float* xb[NB];
    int pos[NB];
    f32x4 y[NB][IB];
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      const int row = (blk0 + p) * 16 + n;
      long long b;
      int sigma;
      tm.decode(row < rows_used ? row : rows_used - 1, b, sigma);  // rows nobody reads: the last one's samples
      pos[p] = (sigma + item.j0) * hop - g.pad + 4 * q;
      xb[p] = EDGE ? g.x + b * g.L : g.x + b * g.L + pos[p];
#pragma unroll
      for (int i = 0; i < IB; ++i) y[p][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    contract(edge_tag, ib_tag, y, xb, pos, P.ub + item.u0 / 2 * 3 + (long long)ib0 * 192, item.n_ib, 0, hop);
    // lane (q, n), register e: row 4 q + e of a basis block, hop-block n.  Block 0's last n_lo rows go to its first.
    const int n_lo = item.n_lo;
    if (ib0 == 0) {
#pragma unroll
      for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = __shfl(y[p][0][e], lane + 64 - 4 * n_lo);  // (in every lane; used by those of the first n_lo rows)
          if (4 * q < n_lo) y[p][0][e] += lo;
        }
    }
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      const int row = (blk0 + p) * 16 + n;
      if (row < rows_used) {
#pragma unroll
        for (int i = 0; i < IB; ++i) {
          const int blk = ib0 + i, f = blk ? 16 * blk - n_lo + 4 * q : 4 * q;
          if (f < r && (blk || f < 16 - n_lo)) {
            if (!split) {
              *reinterpret_cast<f32x4*>(Y + row * r + f) = y[p][i];
            } else {
              const f32x4 both[2] = {y[p][i], y[p][i]};
              const Planes b = split8(both);
#pragma unroll
              for (int l = 0; l < 3; ++l) *reinterpret_cast<uint2*>(Yb + l * p_words + row * r + f) = make_uint2(b.p[l][0], b.p[l][1]);
            }
          }
        }
      }
    }
  };
  {
    // The waves share the (passes over the basis) x (blocks of 16 hop-blocks) evenly, a wave's share in runs of one pass.
    const int nblk = (rows_used + 15) >> 4, n_pass = (item.n_ib + 2) / 3, units = nblk * n_pass;
    const int first = units * wave >> 2, last = units * (wave + 1) >> 2;
    for (int u = first; u < last;) {
      const int pass = u / nblk, blk = u - pass * nblk, todo = (last < (pass + 1) * nblk ? last : (pass + 1) * nblk) - u;
      const int nb = todo <= 4 ? todo : todo <= 6 ? 3 : 4;  // 5 = 3 + 2, 6 = 3 + 3, 7 = 4 + 3
      const int ib = item.n_ib * pass / n_pass, ni = item.n_ib * (pass + 1) / n_pass - ib;  // 1 .. 3 basis blocks
      // does any of these hop-blocks leave its waveform?  lane: one of their (up to 64) rows
      const int row = blk * 16 + lane;
      bool edge = false;
      if (lane < 16 * nb && row < rows_used) {
        long long b;
        int sigma;
        tm.decode(row, b, sigma);
        const int s = (sigma + item.j0) * hop - g.pad;
        edge = s < 0 || s + hop > L;
      }
      auto with_ib = [&](auto edge_tag, auto nb_tag) {
        if (ni == 3) sweep(edge_tag, nb_tag, integral_constant<int, 3>{}, blk, ib);
        else if (ni == 2) sweep(edge_tag, nb_tag, integral_constant<int, 2>{}, blk, ib);
        else sweep(edge_tag, nb_tag, integral_constant<int, 1>{}, blk, ib);
      };
      auto with_nb = [&](auto edge_tag) {
        if (nb == 4) with_ib(edge_tag, integral_constant<int, 4>{});
        else if (nb == 3) with_ib(edge_tag, integral_constant<int, 3>{});
        else if (nb == 2) with_ib(edge_tag, integral_constant<int, 2>{});
        else with_ib(edge_tag, integral_constant<int, 1>{});
      };
      if (__builtin_amdgcn_ballot_w64(edge) != 0) with_nb(True{});
      else with_nb(False{});
      u += nb;
    }
    // the last step of the last frame reads up to 31 words (times zero) past its hop-blocks
    if (tid < 32) {
      if (!split) Y[rows_used * r + tid] = 0.f;
      else
        for (int l = 0; l < 3; ++l) Yb[l * p_words + rows_used * r + tid] = 0;
    }
  }
  __syncthreads();

  // ---- stage 2: the frames' combinations ----------------------------------------------
  clear();
  int y_off[FB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) y_off[fb] = (valid[fb] ? tm.frame_row(wave * (16 * FB) + fb * 16 + n) : 0) * r + 4 * q;
  const uint4* a0p = P.ab + item.a0[0] / 2 * 3 + lane;
  const uint4* a1p = P.ab + item.a0[1] / 2 * 3 - (long long)(item.s_lo / 2) * 192 + lane;
  // steps [s, e) of 32: both row blocks, or the first alone
  auto steps = [&](auto both_tag, auto split_tag, int s, int e) {
    constexpr bool BOTH = decltype(both_tag)::value, SPLIT = decltype(split_tag)::value;
    constexpr int YV = SPLIT ? 3 : 2;  // 16-byte words a step of a frame block takes from LDS
    if (s >= e) return;
    auto fetch = [&](int i, u32x4 (&c0)[3], u32x4 (&c1)[3], u32x4 (&y)[FB][YV]) {
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        c0[l] = *reinterpret_cast<const u32x4*>(a0p + ((long long)i * 3 + l) * 64);
        if constexpr (BOTH) c1[l] = *reinterpret_cast<const u32x4*>(a1p + ((long long)i * 3 + l) * 64);
      }
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int h = 0; h < YV; ++h) {
          if constexpr (SPLIT) {
            const unsigned short* p = Yb + h * p_words + y_off[fb] + 32 * i;
            const uint2 lo = *reinterpret_cast<const uint2*>(p), hi = *reinterpret_cast<const uint2*>(p + 16);
            y[fb][h] = (u32x4){lo.x, lo.y, hi.x, hi.y};
          } else {
            y[fb][h] = *reinterpret_cast<const u32x4*>(Y + y_off[fb] + 32 * i + 16 * h);
          }
        }
    };
    auto multiply = [&](const u32x4 (&c0)[3], const u32x4 (&c1)[3], const u32x4 (&y)[FB][YV]) {
#pragma unroll
      for (int fb = 0; fb < FB; ++fb) {
        Planes b;
        if constexpr (SPLIT) {
#pragma unroll
          for (int l = 0; l < 3; ++l) b.p[l] = y[fb][l];
        } else {
          const f32x4 v[2] = {__builtin_bit_cast(f32x4, y[fb][0]), __builtin_bit_cast(f32x4, y[fb][1])};
          b = split8(v);
        }
        acc[fb][0] += multiply_octets(c0, b, (f32x4){0.f, 0.f, 0.f, 0.f});
        if constexpr (BOTH) acc[fb][1] += multiply_octets(c1, b, (f32x4){0.f, 0.f, 0.f, 0.f});
      }
    };
    // register sets of coefficients and frames, requested up to three steps ahead
    constexpr int SETS = FB == 1 ? 4 : 2;
    u32x4 c0[SETS][3], c1[SETS][3];
    u32x4 y[SETS][FB][YV];
#pragma unroll
    for (int u = 0; u < SETS - 1; ++u) fetch(s + u < e ? s + u : e - 1, c0[u], c1[u], y[u]);
    for (int i = s; i < e; i += SETS) {
#pragma unroll
      for (int u = 0; u < SETS; ++u) {
        const int ahead = i + u + SETS - 1, at = (u + SETS - 1) % SETS;
        fetch(ahead < e ? ahead : e - 1, c0[at], c1[at], y[at]);
        __builtin_amdgcn_sched_barrier(0);
        if (i + u < e) multiply(c0[u], c1[u], y[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto all_steps = [&](auto split_tag) {
    const bool two = item.s_lo < item.s_hi;
    steps(False{}, split_tag, 0, (two ? item.s_lo : item.n_step) / 2);
    if (!two) return;
    steps(True{}, split_tag, item.s_lo / 2, item.s_hi / 2);
    steps(False{}, split_tag, item.s_hi / 2, item.n_step / 2);
  };
  if (split) all_steps(True{});
  else all_steps(False{});
  // A sample that is not finite reaches, through its hop-block's coordinates, bins and frames whose own taps it lies outside of, and
  // turns infinities into NaN.  So a sum that is not finite is taken again over the bin's own taps: those samples alone if there
  // are any, else hop-block by hop-block, the ones whose coordinates are not finite sample by sample.  (1,770 x 176,400 samples, a
  // NaN / an infinity in every waveform: 8.2 -> 320 / 525 ms.)
  unsigned odd = store_bins<FB, RB>(P, item, acc, valid, f0, wave, q, n);
#pragma unroll 1
  while (odd) {
    const int bit = __builtin_ctz(odd), rb = (bit >> 1) % RB, k = 8 * rb + 2 * q + (bit & 1), fi = (wave * FB + (bit >> 1) / RB) * 16 + n;
    odd &= odd - 1;
    const long long f = f0 + fi, b = f / g.T;
    const int t = (int)(f - b * g.T), s0 = rb ? item.s_lo : 0, s1 = rb ? item.s_hi : item.n_step;
    const int2 own = P.support[item.bin0 + k];
    const float* __restrict__ a = reinterpret_cast<const float*>(P.a + (rb ? item.a0[1] : item.a0[0]) + (2 * k & 15));  // (Im: the next row)
    const float* __restrict__ u = reinterpret_cast<const float*>(P.u + item.u0);
    const float* __restrict__ xb = g.x + b * g.L;
    const int y0 = tm.frame_row(fi) * r;
    auto coordinate = [&](int i) {
      if (!split) return Y[y0 + i];
      float v = 0.f;
      for (int l = 2; l >= 0; --l) v += __builtin_bit_cast(float, (unsigned)Yb[l * p_words + y0 + i] << 16);
      return v;
    };
    const int first = own.x / hop - item.j0, last = (own.y - 1) / hop - item.j0;  // hop-blocks of the bin's own taps
    // of hop-block j: its own columns, coefficients of function i, sample and weight of column c
    auto begin = [&](int j) { const int c = own.x - (item.j0 + j) * hop; return c > 0 ? c : 0; };
    auto end = [&](int j) { const int c = own.y - (item.j0 + j) * hop; return c < hop ? c : hop; };
    auto coefficients = [&](int j, int i, float& ar, float& ai) {
      const int w = j * r + i, s = w >> 4, at = ((s - s0) * 64 + ((w >> 2) & 3) * 16) * 4 + (w & 3);
      const bool there = s >= s0 && s < s1;
      ar = there ? a[at] : 0.f;
      ai = there ? a[at + 4] : 0.f;
    };
    auto sample = [&](int j, int c) { return xb[reflect_clamped(t * g.hop - g.pad + (item.j0 + j) * hop + c, L)]; };
    auto weight = [&](int j, int c, float& wr, float& wi) {
      wr = wi = 0.f;
#pragma unroll 1
      for (int i = 0; i < r; ++i) {
        const int at = i < 16 - item.n_lo ? i : i + item.n_lo;  // row of the basis
        const float v = u[((((c >> 5) * item.n_ib + (at >> 4)) * 2 + ((c >> 4) & 1)) * 64 + ((c >> 2) & 3) * 16 + (at & 15)) * 4 + (c & 3)];
        float ar, ai;
        coefficients(j, i, ar, ai);
        wr += ar * v;
        wi += ai * v;
      }
    };
    float re = 0.f, im = 0.f;
    bool met = false;
#pragma unroll 1
    for (int j = first; j <= last; ++j) {
      if (finite(coordinate(j * r))) continue;
#pragma unroll 1
      for (int c = begin(j); c < end(j) && !(re != re && im != im); ++c) {
        const float x = sample(j, c);
        if (finite(x)) continue;
        float wr = 0.f, wi = 0.f;
        if (x == x) weight(j, c, wr, wi);
        re += wr * x;
        im += wi * x;
        met = true;
      }
    }
#pragma unroll 1
    for (int j = first; j <= last && !met; ++j) {
      bool fine = true;
      float yr = 0.f, yi = 0.f;
#pragma unroll 1
      for (int i = 0; i < r; ++i) {
        const float y = coordinate(j * r + i);
        float ar, ai;
        coefficients(j, i, ar, ai);
        fine = fine && finite(y);
        yr += ar * y;
        yi += ai * y;
      }
      if (!fine) {
        yr = yi = 0.f;
#pragma unroll 1
        for (int c = begin(j); c < end(j); ++c) {
          float wr, wi;
          weight(j, c, wr, wi);
          yr += wr * sample(j, c);
          yi += wi * sample(j, c);
        }
      }
      re += yr;
      im += yi;
    }
    store_bin(P.fmt, g.T, P.out + b * P.out_wave_stride + t, item.bin0 + k, re, im);
  }
}

// FB, FD: 16-frame blocks per wave of the items with a basis and of the direct ones.  The direct ones come first, the item the slow
// index; tiles of nna_short.h in their place (SHORT) last, their items neighbours too: they are many and short, those with a basis
// few and long in a short batch (tiles first: 65 us for 46 at 16 x 220,500).  The others: workgroup ids are dealt round-robin to the 8 XCDs, and the items of one tile are neighbours on one XCD,
// where they meet the tile's samples in its L2 (28 million L2 misses instead of 263 million, 7.1 -> 6.5 ms at 1,770 x 176,400);
// rotated by one from tile to tile, because items differ in length and the CUs are dealt out in a fixed order too.
template <int FB, int FD, bool SHORT>
__global__ __launch_bounds__(256, 2) void cqt_lowrank_kernel(const CqlParams P) {
  extern __shared__ __attribute__((aligned(16))) float Y[];
  long long bid = blockIdx.x;
  const long long n_basis = (P.basis.n_ft + 7) / 8 * 8 * P.basis.n_items, n_direct = P.direct.n_ft * P.direct.n_items;
  if (SHORT ? bid >= n_basis : bid < n_direct) {
    if constexpr (SHORT) {
      bid -= n_basis;
      const long long local = bid >> 3, tile = local / P.shorts.n_items, ft = (bid & 7) * ((P.shorts.n_ft + 7) >> 3) + tile;
      if (ft >= P.shorts.n_ft) return;
      const ShortItem item = P.shorts.items[local - tile * P.shorts.n_items];
      short_tile<FD, 4, COLUMNS, 0>(P.shorts, item, ft, reinterpret_cast<unsigned short*>(Y));
    } else {
      const int id = (int)(bid / P.direct.n_ft);
      const CqlItem item = P.direct.items[id];
      direct_item<FD>(P, P.direct, item, bid - (long long)id * P.direct.n_ft, Y);
    }
  } else {
    if (!SHORT) bid -= n_direct;
    const int n_items = P.basis.n_items;
    const long long local = bid >> 3, per_xcd = (P.basis.n_ft + 7) >> 3, tile = local / n_items;
    const long long ft = (bid & 7) * per_xcd + tile;
    if (ft >= P.basis.n_ft) return;
    const CqlItem item = P.basis.items[(local + tile) % n_items];
    lowrank_item<FB>(P, P.basis, item, ft, Y);
  }
}

template <int FB, int FD, bool SHORT = false>
hipError_t allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(cqt_lowrank_kernel<FB, FD, SHORT>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             CQL_LDS_ONE);
}

template <int FB, int FD, bool SHORT = false>
void launch(const CqlParams& p, unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL((cqt_lowrank_kernel<FB, FD, SHORT>), dim3(blocks), dim3(256), (size_t)p.lds_floats * 4, stream, p);
}

}  // namespace

hipError_t cql_kernels_init() {
  hipError_t e = allow_lds<1, 1>();
  if (e == hipSuccess) e = allow_lds<2, 1>();
  if (e == hipSuccess) e = allow_lds<4, 1>();
  if (e == hipSuccess) e = allow_lds<2, 2>();
  if (e == hipSuccess) e = allow_lds<4, 2>();
  if (e == hipSuccess) e = allow_lds<1, 4, true>();
  if (e == hipSuccess) e = allow_lds<2, 4, true>();
  if (e == hipSuccess) e = allow_lds<4, 4, true>();
  return e;
}

hipError_t launch_cqt_lowrank(const CqlParams& p, hipStream_t stream) {
  clear_stale_error();
  const bool shorts = p.shorts.n_items > 0;
  const long long blocks = (p.basis.n_ft + 7) / 8 * 8 * p.basis.n_items +
                           (shorts ? (p.shorts.n_ft + 7) / 8 * 8 * p.shorts.n_items : p.direct.n_ft * p.direct.n_items);
  if (blocks <= 0 || blocks > 0x7fffffffLL || p.g.hop % 32) return hipErrorInvalidValue;
  if (p.basis.tile_frames < 1 || p.basis.tile_frames > 64 * p.basis.fb || p.direct.tile_frames > 64 * p.direct.fb) return hipErrorInvalidValue;
  if (p.lds_floats < 1 || (size_t)p.lds_floats * 4 > (size_t)CQL_LDS_ONE) return hipErrorInvalidValue;
  // (a batch large enough for two blocks per wave of the direct items is so for those with a basis)
  const int fb = p.basis.fb, fd = p.direct.fb;
  if ((fb != 1 && fb != 2 && fb != 4) || (fd != 1 && fd != 2) || fd > fb) return hipErrorInvalidValue;
  if (shorts) {
    const ShortParams& s = p.shorts;
    constexpr int form = SHORT_COLUMNS_64;
    if (s.form != form || s.tile_frames < 1 || s.tile_frames > SHORT_FRAMES[form] || s.plane % 8 != 0 || s.plane < SHORT_PLANE_MIN[form] ||
        s.plane * 6 + 16 > p.lds_floats * 4 || (s.columns_at_once != 32 && s.columns_at_once != 64 && s.columns_at_once != 128) || s.g.L < 4)
      return hipErrorInvalidValue;
    fb == 1 ? launch<1, 4, true>(p, (unsigned)blocks, stream) : fb == 2 ? launch<2, 4, true>(p, (unsigned)blocks, stream) : launch<4, 4, true>(p, (unsigned)blocks, stream);
  } else if (fd == 1)
    fb == 1 ? launch<1, 1>(p, (unsigned)blocks, stream) : fb == 2 ? launch<2, 1>(p, (unsigned)blocks, stream) : launch<4, 1>(p, (unsigned)blocks, stream);
  else
    fb == 2 ? launch<2, 2>(p, (unsigned)blocks, stream) : launch<4, 2>(p, (unsigned)blocks, stream);
  return hipGetLastError();
}

}  // namespace nna
