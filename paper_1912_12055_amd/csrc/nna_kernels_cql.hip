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
// In one launch bound by no one pipe at the batch below: the samples' splits keep the vector ALUs 52 % busy, the matrix pipe is at 39 %; a
// short batch by latency, a workgroup or two per CU.  With a workspace, where that pays, as two: coordinates first, the short kernels beside
// them (pipe 48 % busy, vector ALUs 43 %), then the second stage (62, 59 %).  1,770 x 176,400 samples, 168 bins of 24 per octave (MI355X): 24.5 ms
// folded about the centres, 8.25 here in float32, 6.59 in bfloat16 with every coordinate split by each frame that reads it, now 5.74;
// 16 x 220,500, 84 bins of 12 per octave: 300 -> 67.8 -> 53.8 us; the dense composed kernels of the frequency-domain layer (16 x
// 220,500, 16,384 taps): 566 -> 183 -> 138 us.  With the short kernels by tiles of nna_short.h (the direct items read four row blocks' weights for
// every 16 frames, and the loads' issue bound them): 5.81 -> 5.12 ms, 58 -> 46 us.  In two
// launches: the batch 5.34 -> 4.75 ms, the dense kernels 134 -> 81 us.
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

// Kernels as combinations of the item's basis.  READY: the coordinates are in memory.  SHARED (tiles of 64 frames): the waves share the steps
// of stage 2, each of them for all frames, and their sums are added through LDS at P.shared: every wave reading all weights for 16 frames
// waits for them (16 x 220,500 samples, 84 dense kernels: stage 2 67 -> 50 us).
template <int FB, bool READY, bool SHARED>
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
  const bool split = 6 * p_words <= 4 * (SHARED ? P.shared : P.lds_floats);
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
  if constexpr (READY) {
    // waveform by waveform, the tile's hop-blocks one behind the other as they lie in LDS
    const int quads = r / 4;
    for (int row0 = 0; row0 < rows_used;) {
      long long b;
      int sigma;
      tm.decode(row0, b, sigma);
      const int rows = row0 == 0 ? tm.n0 + tm.extra : tm.T + tm.extra, n_quad = (rows < rows_used - row0 ? rows : rows_used - row0) * quads;
      const f32x4* __restrict__ src = reinterpret_cast<const f32x4*>(P.y + b * P.y_wave + (long long)item.y_r * g.T + item.y_rj) + (long long)sigma * quads;
      constexpr int U = 8;
      for (int i0 = tid; i0 < n_quad; i0 += 256 * U) {
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = src[i0 + 256 * u < n_quad ? i0 + 256 * u : n_quad - 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (i0 + 256 * u >= n_quad) break;
          const int at = row0 * r + 4 * (i0 + 256 * u);
          if (!split) {
            *reinterpret_cast<f32x4*>(Y + at) = v[u];
          } else {
            const f32x4 both[2] = {v[u], v[u]};
            const Planes q3 = split8(both);
#pragma unroll
            for (int l = 0; l < 3; ++l) *reinterpret_cast<uint2*>(Yb + l * p_words + at) = make_uint2(q3.p[l][0], q3.p[l][1]);
          }
        }
      }
      row0 += rows;
    }
  } else {
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
  }
  // the last step of the last frame reads up to 31 words (times zero) past its hop-blocks
  if (tid < 32) {
    if (!split) Y[rows_used * r + tid] = 0.f;
    else
      for (int l = 0; l < 3; ++l) Yb[l * p_words + rows_used * r + tid] = 0;
  }
  __syncthreads();

  // ---- stage 2: the frames' combinations ----------------------------------------------
  static_assert(!SHARED || FB == 1, "a wave ends up with a block of sixteen frames");
  constexpr int MB = SHARED ? 4 : FB;  // frame blocks a wave multiplies
  f32x4 sum[MB][RB];
  int y_off[MB];
#pragma unroll
  for (int fb = 0; fb < MB; ++fb) {
    const int fi = SHARED ? fb * 16 + n : wave * (16 * FB) + fb * 16 + n;
    y_off[fb] = (fi < m_valid ? tm.frame_row(fi) : 0) * r + 4 * q;
#pragma unroll
    for (int b = 0; b < RB; ++b) sum[fb][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const uint4* a0p = P.ab + item.a0[0] / 2 * 3 + lane;
  const uint4* a1p = P.ab + item.a0[1] / 2 * 3 - (long long)(item.s_lo / 2) * 192 + lane;
  // steps [s, e) of 32: both row blocks, or the first alone
  auto steps = [&](auto both_tag, auto split_tag, int s, int e) {
    constexpr bool BOTH = decltype(both_tag)::value, SPLIT = decltype(split_tag)::value;
    constexpr int YV = SPLIT ? 3 : 2;  // 16-byte words a step of a frame block takes from LDS
    if constexpr (SHARED) s += wave;
    if (s >= e) return;
    constexpr int BY = SHARED ? 4 : 1;
    auto fetch = [&](int i, u32x4 (&c0)[3], u32x4 (&c1)[3], u32x4 (&y)[MB][YV]) {
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        c0[l] = *reinterpret_cast<const u32x4*>(a0p + ((long long)i * 3 + l) * 64);
        if constexpr (BOTH) c1[l] = *reinterpret_cast<const u32x4*>(a1p + ((long long)i * 3 + l) * 64);
      }
#pragma unroll
      for (int fb = 0; fb < MB; ++fb)
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
    auto multiply = [&](const u32x4 (&c0)[3], const u32x4 (&c1)[3], const u32x4 (&y)[MB][YV]) {
#pragma unroll
      for (int fb = 0; fb < MB; ++fb) {
        Planes b;
        if constexpr (SPLIT) {
#pragma unroll
          for (int l = 0; l < 3; ++l) b.p[l] = y[fb][l];
        } else {
          const f32x4 v[2] = {__builtin_bit_cast(f32x4, y[fb][0]), __builtin_bit_cast(f32x4, y[fb][1])};
          b = split8(v);
        }
        sum[fb][0] += multiply_octets(c0, b, (f32x4){0.f, 0.f, 0.f, 0.f});
        if constexpr (BOTH) sum[fb][1] += multiply_octets(c1, b, (f32x4){0.f, 0.f, 0.f, 0.f});
      }
    };
    // register sets of coefficients and frames, requested up to three steps ahead
    constexpr int SETS = MB == 1 ? 4 : 2;
    u32x4 c0[SETS][3], c1[SETS][3];
    u32x4 y[SETS][MB][YV];
#pragma unroll
    for (int u = 0; u < SETS - 1; ++u) fetch(s + BY * u < e ? s + BY * u : s, c0[u], c1[u], y[u]);
    for (int i = s; i < e; i += BY * SETS) {
#pragma unroll
      for (int u = 0; u < SETS; ++u) {
        const int ahead = i + BY * (u + SETS - 1), at = (u + SETS - 1) % SETS;
        fetch(ahead < e ? ahead : s, c0[at], c1[at], y[at]);
        __builtin_amdgcn_sched_barrier(0);
        if (i + BY * u < e) multiply(c0[u], c1[u], y[u]);
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
  if constexpr (SHARED) {
    // wave k takes frame block k: the other waves' sums in their order, then its own
    f32x4* const part = reinterpret_cast<f32x4*>(Y + P.shared) + lane;  // [frame block][three waves][row block][64 lanes]
#pragma unroll
    for (int fb = 0; fb < MB; ++fb) {
      if (fb == wave) continue;
#pragma unroll
      for (int b = 0; b < RB; ++b) part[((fb * 3 + (wave < fb ? wave : wave - 1)) * RB + b) * 64] = sum[fb][b];
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      acc[0][b] = part[(wave * 3 * RB + b) * 64];
      acc[0][b] += part[((wave * 3 + 1) * RB + b) * 64];
      acc[0][b] += part[((wave * 3 + 2) * RB + b) * 64];
#pragma unroll
      for (int fb = 0; fb < MB; ++fb)
        if (fb == wave) acc[0][b] += sum[fb][b];
    }
  } else {
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
      for (int b = 0; b < RB; ++b) acc[fb][b] = sum[fb][b];
  }
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

// tile `bid` of the short kernels
template <int FD>
__device__ __forceinline__ void short_work(const CqlParams& P, long long bid, float* Y) {
  const long long local = bid >> 3, tile = local / P.shorts.n_items, ft = (bid & 7) * ((P.shorts.n_ft + 7) >> 3) + tile;
  if (ft >= P.shorts.n_ft) return;
  const ShortItem item = P.shorts.items[local - tile * P.shorts.n_items];
  short_tile<FD, 4, COLUMNS, 0>(P.shorts, item, ft, reinterpret_cast<unsigned short*>(Y));
}

// FB, FD: 16-frame blocks per wave of the items with a basis and of the direct ones.  The direct ones come first, the item the slow
// index; tiles of nna_short.h in their place (SHORT) last, their items neighbours too: they are many and short, those with a basis
// few and long in a short batch (tiles first: 65 us for 46 at 16 x 220,500).  The others: workgroup ids are dealt round-robin to the 8 XCDs, and the items of one tile are neighbours on one XCD,
// where they meet the tile's samples in its L2 (28 million L2 misses instead of 263 million, 7.1 -> 6.5 ms at 1,770 x 176,400);
// rotated by one from tile to tile, because items differ in length and the CUs are dealt out in a fixed order too.
template <int FB, int FD, bool SHORT, bool READY, bool SHARED>
__global__ __launch_bounds__(256, 2) void cqt_lowrank_kernel(const CqlParams P) {
  extern __shared__ __attribute__((aligned(16))) float Y[];
  long long bid = blockIdx.x;
  const long long n_basis = (P.basis.n_ft + 7) / 8 * 8 * P.basis.n_items, n_direct = P.direct.n_ft * P.direct.n_items;
  if (SHORT ? bid >= n_basis : bid < n_direct) {
    if constexpr (SHORT) {
      short_work<FD>(P, bid - n_basis, Y);
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
    lowrank_item<FB, READY, SHARED>(P, P.basis, item, ft, Y);
  }
}

__device__ __host__ inline long long g_rows(const CqlParams& P) { return P.g.B * P.y_rows; }

// Stage 1 by itself: every hop-block's coordinates of all items, once.  A workgroup takes 16 NB hop-blocks and a part of the bases' row
// blocks; the samples are split once, on the way into LDS, 64 columns at a time, and each wave multiplies every fourth row block with all
// of them, so that a workgroup reads its weights once.  The sums are those of lowrank_item, in the same order.  lowrank_item itself reads and
// splits every sample for each 16 bins, and for every tile whose frames reach it: 2.2 ms of 5.34 at 1,770 x 176,400 samples, 168 bins; here 1.5 ms
// (41 % of the matrix pipe's peak; weights from the L2s at 31 bytes a cycle and CU), the call 4.75.  16 x 220,500, 84 dense kernels of
// 16,384 taps: 137 -> 86 us, of which 33 here.
constexpr int PJ_COLS = 64, PJ_PITCH = PJ_COLS + 8;  // (rows of 36 words: sixteen of them on different banks, four words each)
constexpr int PJ_LDS(int nb) { return 2 * 3 * 16 * nb * PJ_PITCH * 2; }

template <int NB, int IB, bool SHORT>
__global__ __launch_bounds__(256, 2) void cqt_project_kernel(const CqlParams P) {
  extern __shared__ __attribute__((aligned(16))) float Y[];
  if constexpr (SHORT) {
    const long long n_project = ((g_rows(P) + 16 * NB - 1) / (16 * NB) + 7) / 8 * 8 * P.y_groups;
    if (blockIdx.x >= n_project) {
      short_work<4>(P, blockIdx.x - n_project, Y);
      return;
    }
  }
  unsigned short* const S = reinterpret_cast<unsigned short*>(Y);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int q = lane >> 4, n = lane & 15;
  const FrameGeom& g = P.g;
  const int L = (int)g.L, hop = g.hop;
  constexpr int ROWS = 16 * NB, PLANE = ROWS * PJ_PITCH, UNITS = NB / 2;
  // neighbouring tiles, and the parts of one, on one XCD, whose L2 they share
  const long long n_rows = g_rows(P), n_tiles = (n_rows + ROWS - 1) / ROWS, per_xcd = (n_tiles + 7) >> 3;
  const long long local = blockIdx.x >> 3, in_xcd = local / P.y_groups, tile = (blockIdx.x & 7) * per_xcd + in_xcd;
  const int group = (int)(local - in_xcd * P.y_groups);
  if (in_xcd >= per_xcd || tile >= n_tiles) return;
  const long long row_first = tile * ROWS, b_first = row_first / P.y_rows;
  const int s_first = (int)(row_first - b_first * P.y_rows);
  auto decode = [&](int i, long long& b, int& s) {  // hop-block i of the tile; behind the last one: that one
    if (row_first + i >= n_rows) i = (int)(n_rows - 1 - row_first);
    const int u = s_first + i, w = u < P.y_rows ? 0 : u / P.y_rows;
    b = b_first + w;
    s = u - w * P.y_rows;
  };
  // this wave's row blocks: item, and block of its basis (behind the last: that one, not written)
  const int blk0 = P.y_blocks * group / P.y_groups, blk1 = P.y_blocks * (group + 1) / P.y_groups;
  int item_of[IB], ib_of[IB], stride[IB];
  const uint4* up[IB];
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    int rb = blk0 + wave + 4 * i < blk1 ? blk0 + wave + 4 * i : blk1 - 1, it = 0;
    while (rb >= P.basis.items[it].n_ib) rb -= P.basis.items[it++].n_ib;
    item_of[i] = it;
    ib_of[i] = rb;
    stride[i] = P.basis.items[it].n_ib * 192;
    up[i] = P.ub + P.basis.items[it].u0 / 2 * 3 + rb * 192 + lane;
  }
  // this thread's octets of a chunk: four columns and the four sixteen behind them
  const float* xb[UNITS];
  int pos[UNITS];
  bool edge = false;
#pragma unroll
  for (int k = 0; k < UNITS; ++k) {
    const int o = tid + 256 * k;
    long long b;
    int s;
    decode(o >> 3, b, s);
    const int first = (s + P.y_j0) * hop - g.pad;
    xb[k] = g.x + b * g.L;
    pos[k] = first + (o >> 2 & 1) * 32 + (o & 3) * 4;
    edge = edge || first < 0 || first + hop > L;
  }
  const bool wave_edge = __builtin_amdgcn_ballot_w64(edge) != 0;
  const bool second = (tid >> 2 & 1) != 0;  // the chunk's second 32 columns, which a hop's last one may lack
  f32x4 v[UNITS][2];
  auto request = [&](int c) {
    if (second && c + 32 >= hop) return;
    if (!wave_edge) {
#pragma unroll
      for (int k = 0; k < UNITS; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) v[k][h] = *reinterpret_cast<const f32x4_u*>(xb[k] + pos[k] + c + 16 * h);
    } else {
#pragma unroll
      for (int k = 0; k < UNITS; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int s = pos[k] + c + 16 * h, src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
          if ((unsigned)src <= (unsigned)(L - 4)) {
            const f32x4 t = *reinterpret_cast<const f32x4_u*>(xb[k] + src);
            v[k][h] = src != s ? (f32x4){t.w, t.z, t.y, t.x} : t;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[k][h][e] = xb[k][reflect_clamped(s + e, L)];
          }
        }
    }
  };
  auto put = [&](int c, unsigned short* dst) {
    if (second && c + 32 >= hop) return;
#pragma unroll
    for (int k = 0; k < UNITS; ++k) {
      const int o = tid + 256 * k;
      const Planes b = split8(v[k]);
#pragma unroll
      for (int l = 0; l < 3; ++l) *reinterpret_cast<u32x4*>(dst + l * PLANE + (o >> 3) * PJ_PITCH + (o & 7) * 8) = b.p[l];
    }
  };
  f32x4 acc[NB][IB];
#pragma unroll
  for (int p = 0; p < NB; ++p)
#pragma unroll
    for (int i = 0; i < IB; ++i) acc[p][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int n_step = hop / 32;
  u32x4 w[2][3];
  auto fetch_w = [&](int i, int step, u32x4 (&to)[3]) {
    const uint4* from = up[i] + (long long)(step < n_step ? step : n_step - 1) * stride[i];
#pragma unroll
    for (int l = 0; l < 3; ++l) to[l] = *reinterpret_cast<const u32x4*>(from + l * 64);
  };
  request(0);
  fetch_w(0, 0, w[0]);
  put(0, S);
  for (int c = 0; c < hop; c += PJ_COLS) {
    unsigned short* const tile_c = S + (c / PJ_COLS & 1) * 3 * PLANE;
    __syncthreads();  // also: the other buffer has been read by every wave
    if (c + PJ_COLS < hop) request(c + PJ_COLS);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (c + 32 * h >= hop) break;
      Planes x[NB];
#pragma unroll
      for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int l = 0; l < 3; ++l) x[p].p[l] = *reinterpret_cast<const u32x4*>(tile_c + l * PLANE + (16 * p + n) * PJ_PITCH + 32 * h + 8 * q);
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        constexpr int PARITY = IB & 1;
        const int set = (i + h * PARITY) & 1;
        fetch_w(i + 1 < IB ? i + 1 : 0, c / 32 + h + (i + 1 < IB ? 0 : 1), w[set ^ 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < NB; ++p) acc[p][i] += multiply_octets(w[set], x[p], (f32x4){0.f, 0.f, 0.f, 0.f});
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (c + PJ_COLS < hop) put(c + PJ_COLS, S + (c / PJ_COLS + 1 & 1) * 3 * PLANE);
  }
  // lane (q, n), register e: row 4 q + e of a basis block, hop-block n.  Block 0's last n_lo rows go to its first.
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    if (blk0 + wave + 4 * i >= blk1) break;
    const CqlItem& item = P.basis.items[item_of[i]];
    const int n_lo = item.n_lo, ib = ib_of[i], r = item.r, rows = g.T + item.jspan - 1, f = ib ? 16 * ib - n_lo + 4 * q : 4 * q;
    if (ib == 0) {
#pragma unroll
      for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = __shfl(acc[p][i][e], lane + 64 - 4 * n_lo);  // (in every lane; used by those of the first n_lo rows)
          if (4 * q < n_lo) acc[p][i][e] += lo;
        }
    }
    if (f >= r || (!ib && f >= 16 - n_lo)) continue;
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      long long b;
      int s;
      decode(16 * p + n, b, s);
      s -= item.j0 - P.y_j0;
      if (row_first + 16 * p + n < n_rows && s >= 0 && s < rows)
        *reinterpret_cast<f32x4*>(P.y + b * P.y_wave + (long long)item.y_r * g.T + item.y_rj + (long long)s * r + f) = acc[p][i];
    }
  }
}

template <typename K>
hipError_t allow(K kernel) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, CQL_LDS_ONE);
}
template <int FB, int FD, bool SHORT>
hipError_t allow_lds() {
  return allow(cqt_lowrank_kernel<FB, FD, SHORT, false, false>);
}
template <int FB, int FD, bool SHARED>
hipError_t allow_ready() {
  return allow(cqt_lowrank_kernel<FB, FD, false, true, SHARED>);
}
template <int NB, int IB>
hipError_t allow_project() {
  const hipError_t e = allow(cqt_project_kernel<NB, IB, false>);
  return e == hipSuccess ? allow(cqt_project_kernel<NB, IB, true>) : e;
}

template <int FB, int FD, bool SHORT = false>
void launch(const CqlParams& p, unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL((cqt_lowrank_kernel<FB, FD, SHORT, false, false>), dim3(blocks), dim3(256), (size_t)p.lds_floats * 4, stream, p);
}
// stage 2 of the items with a basis (and direct items), their coordinates in memory
template <int FB, int FD, bool SHARED>
void launch_ready(const CqlParams& p, unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL((cqt_lowrank_kernel<FB, FD, false, true, SHARED>), dim3(blocks), dim3(256), (size_t)p.lds_floats * 4, stream, p);
}

template <int NB, int IB>
void launch_project(const CqlParams& p, hipStream_t stream) {
  const long long n_project = ((g_rows(p) + 16 * NB - 1) / (16 * NB) + 7) / 8 * 8 * p.y_groups;
  if (p.shorts.n_items) {
    const size_t lds = (size_t)p.shorts.plane * 6 + 16;
    hipLaunchKernelGGL((cqt_project_kernel<NB, IB, true>), dim3((unsigned)(n_project + (p.shorts.n_ft + 7) / 8 * 8 * p.shorts.n_items)), dim3(256),
                       lds < PJ_LDS(NB) ? PJ_LDS(NB) : lds, stream, p);
  } else {
    hipLaunchKernelGGL((cqt_project_kernel<NB, IB, false>), dim3((unsigned)n_project), dim3(256), PJ_LDS(NB), stream, p);
  }
}

}  // namespace

hipError_t cql_kernels_init() {
  hipError_t e = allow_lds<1, 1, false>();
  if (e == hipSuccess) e = allow_lds<2, 1, false>();
  if (e == hipSuccess) e = allow_lds<4, 1, false>();
  if (e == hipSuccess) e = allow_lds<2, 2, false>();
  if (e == hipSuccess) e = allow_lds<4, 2, false>();
  if (e == hipSuccess) e = allow_lds<1, 4, true>();
  if (e == hipSuccess) e = allow_lds<2, 4, true>();
  if (e == hipSuccess) e = allow_lds<4, 4, true>();
  if (e == hipSuccess) e = allow_ready<1, 1, false>();
  if (e == hipSuccess) e = allow_ready<1, 1, true>();
  if (e == hipSuccess) e = allow_ready<2, 1, false>();
  if (e == hipSuccess) e = allow_ready<4, 1, false>();
  if (e == hipSuccess) e = allow_ready<2, 2, false>();
  if (e == hipSuccess) e = allow_ready<4, 2, false>();
  if (e == hipSuccess) e = allow_project<2, 3>();
  if (e == hipSuccess) e = allow_project<4, 3>();
  if (e == hipSuccess) e = allow_project<2, 6>();
  if (e == hipSuccess) e = allow_project<4, 6>();
  return e;
}

static bool short_fits(const CqlParams& p, size_t lds) {
  const ShortParams& s = p.shorts;
  constexpr int form = SHORT_COLUMNS_64;
  return s.form == form && s.tile_frames >= 1 && s.tile_frames <= SHORT_FRAMES[form] && s.plane % 8 == 0 && s.plane >= SHORT_PLANE_MIN[form] &&
         (size_t)s.plane * 6 + 16 <= lds && (s.columns_at_once == 32 || s.columns_at_once == 64 || s.columns_at_once == 128) && s.g.L >= 4;
}

// Stage 1 of p's items, to p.y, and the short kernels' tiles
hipError_t launch_cqt_project(const CqlParams& p, hipStream_t stream) {
  clear_stale_error();
  if (!p.y || p.basis.n_items < 1 || p.g.hop % 32 || p.y_rows < 1 || p.y_groups < 1 || p.y_blocks < p.y_groups) return hipErrorInvalidValue;
  const int each = (p.y_blocks + p.y_groups - 1) / p.y_groups;  // row blocks of a workgroup
  if (each > 24 || (p.y_nb != 2 && p.y_nb != 4) || (p.shorts.n_items && !short_fits(p, CQL_LDS_ONE)) || (p.g.B * p.y_rows / (16 * p.y_nb) + 8) * p.y_groups > 0x7fffffffLL) return hipErrorInvalidValue;
  if (each <= 12)
    p.y_nb == 2 ? launch_project<2, 3>(p, stream) : launch_project<4, 3>(p, stream);
  else
    p.y_nb == 2 ? launch_project<2, 6>(p, stream) : launch_project<4, 6>(p, stream);
  return hipGetLastError();
}

hipError_t launch_cqt_lowrank(const CqlParams& p, hipStream_t stream) {
  clear_stale_error();
  const bool shorts = p.shorts.n_items > 0 && !p.y;  // (coordinates in memory: the launch before this one took them)
  const long long blocks = (p.basis.n_ft + 7) / 8 * 8 * p.basis.n_items +
                           (shorts ? (p.shorts.n_ft + 7) / 8 * 8 * p.shorts.n_items : p.direct.n_ft * p.direct.n_items);
  if (blocks <= 0 || blocks > 0x7fffffffLL || p.g.hop % 32) return hipErrorInvalidValue;
  if (p.basis.tile_frames < 1 || p.basis.tile_frames > 64 * p.basis.fb || p.direct.tile_frames > 64 * p.direct.fb) return hipErrorInvalidValue;
  if (p.lds_floats < 1 || (size_t)p.lds_floats * 4 > (size_t)CQL_LDS_ONE) return hipErrorInvalidValue;
  // (a batch large enough for two blocks per wave of the direct items is so for those with a basis)
  const int fb = p.basis.fb, fd = p.direct.fb;
  if ((fb != 1 && fb != 2 && fb != 4) || (fd != 1 && fd != 2) || fd > fb) return hipErrorInvalidValue;
  if (p.y) {
    const unsigned n = (unsigned)blocks;
    if (fb == 1)
      p.shared ? launch_ready<1, 1, true>(p, n, stream) : launch_ready<1, 1, false>(p, n, stream);
    else if (fd == 1)
      fb == 2 ? launch_ready<2, 1, false>(p, n, stream) : launch_ready<4, 1, false>(p, n, stream);
    else
      fb == 2 ? launch_ready<2, 2, false>(p, n, stream) : launch_ready<4, 2, false>(p, n, stream);
  } else if (shorts) {
    if (!short_fits(p, (size_t)p.lds_floats * 4)) return hipErrorInvalidValue;
    fb == 1 ? launch<1, 4, true>(p, (unsigned)blocks, stream) : fb == 2 ? launch<2, 4, true>(p, (unsigned)blocks, stream) : launch<4, 4, true>(p, (unsigned)blocks, stream);
  } else if (fd == 1)
    fb == 1 ? launch<1, 1>(p, (unsigned)blocks, stream) : fb == 2 ? launch<2, 1>(p, (unsigned)blocks, stream) : launch<4, 1>(p, (unsigned)blocks, stream);
  else
    fb == 2 ? launch<2, 2>(p, (unsigned)blocks, stream) : launch<4, 2>(p, (unsigned)blocks, stream);
  return hipGetLastError();
}

}  // namespace nna
