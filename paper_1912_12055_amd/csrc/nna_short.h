// Constant-Q transform with time-domain kernels (Sec. III-C, eq. (CQT)), tap by tap: the octaves of the downsampling layers, whose
// kernels are short and whose hops are small.
//
//     C_k[t] = sum_n w_k[n] x[t hop + n]
//
// On v_mfma_f32_16x16x32_bf16, every float32 as three bfloat16 and six products of nine (see nna_kernels_cql.hip, which takes its sums
// the same way: 32 products from zero, then added to a total).  A workgroup takes one item -- up to 24 neighbouring bins, three blocks of
// 16 rows -- and one tile of frames.  Neighbouring frames share most of their samples, so samples are split once, on the way into LDS,
// and every step of 32 taps finds its operand there as it goes into the instruction.  Kernels shrink from row block to row block: a step
// knows how many of them it has taps of.
//   Tiles of 64, 32 or 16 frames: all their samples at once, one behind the other; each wave takes every fourth step of all frames, so
//   that a workgroup reads the weights once, and the waves' sums are added through LDS.
// A tile's rows are whole hops, which neighbouring frames share, or every frame's own taps, where these are fewer than a hop's.
//   Tiles of 128 frames, where 64 frames' samples do not fit: 32 columns of all their rows at a time, the next 32
//   requested while the last step of these is multiplied (loads return in order: requested earlier, they would be waited for with the
//   next step's weights).
//   Tiles of 64 frames by columns: up to 128 at a time, the steps shared as above; kernels of many hops, and those beside the items with a
//   basis of nna_kernels_cql.hip.
//
// Bound by the matrix pipe and the splits in turn while hops are short (hop 64: pipe 58 % busy, vector ALUs 62 %, three workgroups per CU),
// by latency where a tile is read column by column (hop 512: 26 %, 48 %).  1,770 x 345 frames, 24 bins of up to 742 taps
// (MI355X), hop 512 down to 8, against cqt_kernel's float32 instruction:
//   683, 494, 484, 359, 312, 292, 325 us -> 398, 306, 267, 196, 193, 183, 177;
// 16 x 431 frames, 12 bins: 30, 29, 23, 17, 15, 14, 14 -> 10, 9, 10, 8, 9, 9, 9.  (hop 512 and 256 with the samples read straight into
// registers by every wave: 527, 459 us; with tiles of 256 frames by columns, two workgroups per CU: 512, 375; hop 64 by columns: 233.)
// Errors against 64 bits, 2-norm: 5e-8 .. 1.8e-7 of an octave where cqt_kernel's chains are off by 2.5e-7 .. 8e-7.
#pragma once

#include "nna_device.h"

namespace nna {
namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef f32x4 f32x4_u __attribute__((aligned(4)));

// Samples are multiplied by 2^10 before they are split: the third bfloat16 of those below 2^-110 would lose bits to the exponent's end.  An
// octave's error, 2-norm of its worst bin, samples of 1e-34, 1e-36, 1e-38: 3.8e-7 .. 1.2e-6, 6e-7 .. 9e-6, 6e-5 .. 9e-4 with
// cqt_kernel's float32 instruction, 1.1e-6, 1.0e-4, 1.1e-2 as they are, 0.9e-7 .. 1.8e-7, 1.4e-7 .. 2.6e-7, 1.0e-5 .. 1.8e-5.  (By 2^24, 3e-6 ..
// 1.5e-5 at 1e-38, but samples above 2e31 would be none that bfloat16 holds.)  Octaves only: kernels beside a basis are as exact as those with
// one either way, and 16 x 220,500 samples, 84 bins, took 41.0 us for 41.7.
constexpr int SHORT_SCALE = 10;
// the first bfloat16 of 2^SCALE v is finite
template <int SCALE>
__device__ __forceinline__ bool tame(float v) { return (__builtin_bit_cast(unsigned, v) & 0x7fffffffu) < 0x7f7f8000u - ((unsigned)SCALE << 23); }

// where a tile's samples lie in LDS: one behind the other, in words of eight or (rows that are no multiple of 8) of four; or some columns of
// all its rows at a time
enum { OCTETS_OF, QUADS_OF, COLUMNS };

// WK = 4: the four waves share the steps of 16 FB frames; 1: each has 16 FB frames of its own.
template <int FB, int WK, int LAYOUT, int SCALE>
__device__ __forceinline__ void short_tile(const ShortParams& P, const ShortItem& item, long long ft, unsigned short* S) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int q = lane >> 4, n = lane & 15;
  const FrameGeom& g = P.g;
  const long long f0 = ft * P.tile_frames;
  const int m_valid = (int)((g.n_frames - f0) < P.tile_frames ? (g.n_frames - f0) : P.tile_frames);
  TileMap tm;
  tm.T = g.T;
  tm.b0 = f0 / g.T;
  tm.t0 = (int)(f0 - tm.b0 * g.T);
  tm.n0 = (g.T - tm.t0) < m_valid ? (g.T - tm.t0) : m_valid;
  tm.extra = item.jspan - 1;
  const int rows_used = tm.frame_row(m_valid - 1) + tm.extra + 1;
  const int hop = g.hop, width = item.width, L = (int)g.L;
  constexpr int RB = SHORT_RB, THREADS = 256;
  constexpr bool OCTETS = LAYOUT == OCTETS_OF;
  const int plane = P.plane;  // values per plane
  const int n_step = item.n_step;
  const int* __restrict__ steps = P.steps + item.step0;  // row blocks with taps
  const uint4* __restrict__ wp = P.w + item.w0 + lane;   // [step][row block][3 planes][64 lanes]
  auto fetch_w = [&](int s, u32x4 (&v)[RB][3]) {
    const int at = s < n_step ? s : n_step - 1;  // (what is behind the last is read and dropped)
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int l = 0; l < 3; ++l) v[i][l] = *reinterpret_cast<const u32x4*>(wp + ((at * RB + i) * 3 + l) * 64);
  };
  const int wf = wave / WK, wk = wave % WK;
  u32x4 w[RB][3];

  // ---- samples: split once, on the way into LDS ----------------------------------------------
  // A sample that is not finite, or so large that its first bfloat16 is not, would make every sum that holds its step of 32 taps NaN.  It
  // counts as zero here, and its products are added to the bins whose own taps meet it at the end.
  int* const flag = reinterpret_cast<int*>(S + 3 * plane);
  if (tid == 0) *flag = 0;
  __syncthreads();
  auto reflect_run = [&](int s) { return s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s; };
  // four samples from `s` of waveform xb on: a stored run, read backwards behind an end; one that straddles an end sample by sample
  auto four = [&](const float* __restrict__ xb, int s) {
    f32x4 v;
    const int src = reflect_run(s);
    if ((unsigned)src <= (unsigned)(L - 4)) {
      v = *reinterpret_cast<const f32x4_u*>(xb + src);
      if (src != s) v = (f32x4){v.w, v.z, v.y, v.x};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = xb[reflect_clamped(s + e, L)];
    }
    return v;
  };
  // a unit's parts; `v` may change
  auto planes = [&](f32x4 (&v)[2]) {
    v[0] *= (float)(1 << SCALE);
    if constexpr (LAYOUT != QUADS_OF) v[1] *= (float)(1 << SCALE);
    else v[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    Planes b = split8(v);
    u16x2 top = {0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, b.p[0][i] & 0x7fff7fffu));
    if (__builtin_expect(__builtin_elementwise_max(top.x, top.y) >= 0x7f80, 0)) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[h][e] = tame<0>(v[h][e]) ? v[h][e] : 0.f;
      b = split8(v);
      *flag = 1;
    }
    return b;
  };
  constexpr int EB = WK == 1 ? FB : 1;  // frame blocks a wave ends up with
  f32x4 acc[EB][RB], sum[FB][RB];
  int x_off[FB];
#pragma unroll
  for (int fb = 0; fb < FB; ++fb) {
    const int i = wf * (16 * FB) + fb * 16 + n;
    x_off[fb] = (i < m_valid ? tm.frame_row(i) : 0) * (LAYOUT == COLUMNS ? (WK == 1 ? 32 : P.columns_at_once) + 8 : width) + 8 * q;
#pragma unroll
    for (int b = 0; b < RB; ++b) sum[fb][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  // one octet of every nine is left free, so that frames whose rows are 16 .. 512 apart lie on different banks
  auto place = [](int i) { return OCTETS ? i + (i >> 6 << 3) : i; };
  // a step whose first value is `offset` from the frame's row, for its first `a` row blocks; each block's weights make room for step `next`'s
  auto step = [&](int a, int offset, int next) {
    u32x4 x[FB][3];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      const unsigned short* p = S + place(x_off[fb] + offset);
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        if constexpr (LAYOUT != QUADS_OF) {
          x[fb][l] = *reinterpret_cast<const u32x4*>(p + l * plane);
        } else {
          const uint2 lo = *reinterpret_cast<const uint2*>(p + l * plane), hi = *reinterpret_cast<const uint2*>(p + l * plane + 4);
          x[fb][l] = (u32x4){lo.x, lo.y, hi.x, hi.y};
        }
      }
    }
    constexpr int lw[6] = {2, 1, 0, 1, 0, 0}, lx[6] = {0, 1, 2, 0, 1, 0};  // (small terms first)
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      if (i < a) {
        f32x4 t[FB];
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) t[fb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
          for (int fb = 0; fb < FB; ++fb)
            t[fb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[i][lw[m]]), __builtin_bit_cast(bf16x8, x[fb][lx[m]]), t[fb], 0, 0, 0);
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) sum[fb][i] += t[fb];
      }
#pragma unroll
      for (int l = 0; l < 3; ++l) w[i][l] = *reinterpret_cast<const u32x4*>(wp + ((next * RB + i) * 3 + l) * 64);
    }
  };
  if constexpr (LAYOUT == COLUMNS) {
    constexpr int NP = WK == 1 ? FB : SHORT_PASSES;
    const int kc = WK == 1 ? 32 : P.columns_at_once, pitch = kc + 8;  // (rows of 16 frames then lie on different banks)
    // this thread's eight columns of every so many-th row
    const int per_row = kc / 8, cv = tid & (per_row - 1), r0 = tid / per_row, rows_pass = THREADS / per_row;
    const float* xb[NP];
    int pos[NP];
    bool edge[NP];  // does a row of the wave leave its waveform?
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int row = p * rows_pass + r0;
      long long b;
      int sigma;
      tm.decode(row < rows_used ? row : rows_used - 1, b, sigma);
      xb[p] = g.x + b * g.L;
      pos[p] = sigma * hop + item.base - g.pad + 8 * cv;
      edge[p] = __builtin_amdgcn_ballot_w64(pos[p] < 0 || pos[p] > L - ((width + kc - 1) & -kc)) != 0;
      if (!edge[p]) xb[p] += pos[p];
    }
    f32x4 R[NP][2];
    auto request = [&](int c) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (WK > 1 && p * rows_pass >= rows_used) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (!edge[p]) {
            R[p][h] = *reinterpret_cast<const f32x4_u*>(xb[p] + c + 4 * h);
          } else {
            const int src = reflect_run(pos[p] + c + 4 * h);
            R[p][h] = *reinterpret_cast<const f32x4_u*>(xb[p] + (src < 0 ? 0 : src > L - 4 ? L - 4 : src));
          }
        }
      }
    };
    // how many steps lie ahead of every 32 columns, [width / 32 + 1], then the steps in that order: row blocks | row << 2 | which 32
    // columns << 12; step
    const int* __restrict__ ahead_of = P.columns + item.columns;
    const int2* __restrict__ order = reinterpret_cast<const int2*>(ahead_of + (width / 32 + 2) / 2 * 2);
    const int n_order = ahead_of[width / 32];
    int at = wk;
    int2 d = order[at < n_order ? at : 0];
    fetch_w(d.y, w);
    request(0);
    for (int c = 0; c < width; c += kc) {
      __syncthreads();  // the columns before have been read by every wave
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int row = p * rows_pass + r0;
        if (row >= rows_used) continue;
        f32x4 v[2] = {R[p][0], R[p][1]};
#pragma unroll
        for (int h = 0; h < 2 && edge[p]; ++h) {
          const int s = pos[p] + c + 4 * h, src = reflect_run(s);
          if (src != s) v[h] = (f32x4){v[h].w, v[h].z, v[h].y, v[h].x};
          if ((unsigned)src > (unsigned)(L - 4)) v[h] = four(xb[p], s);
        }
        const Planes b = planes(v);
#pragma unroll
        for (int l = 0; l < 3; ++l) *reinterpret_cast<u32x4*>(S + l * plane + row * pitch + 8 * cv) = b.p[l];
      }
      __syncthreads();
      // (loads return in order: the next columns are requested behind the weights of these columns' last step)
      const int end = ahead_of[(c + kc < width ? c + kc : width) / 32], next_c = c + kc < width ? c + kc : c;
      if (at >= end) request(next_c);
      for (; at < end; at += WK) {
        if (at + WK >= end) request(next_c);
        const int2 dn = order[at + WK < n_order ? at + WK : at];
        step(d.x & 3, (d.x >> 2 & 1023) * pitch + 32 * (d.x >> 12 & (kc / 32 - 1)), dn.y);
        d = dn;
      }
    }
  } else {
    fetch_w(wk, w);
    constexpr int N = OCTETS ? 8 : 4, U = 4;  // samples of a unit, units a thread requests at a time
    const int per_row = width / N, units = rows_used * per_row, first = tm.n0 + tm.extra, seg = g.T + tm.extra;
    const float inv_row = 1.f / (float)per_row, inv_seg = 1.f / (float)seg;
    const int base = item.base - g.pad;
    const float* __restrict__ x0 = g.x + tm.b0 * g.L;
    for (int u0 = tid; u0 < units + 32 / N; u0 += THREADS * U) {
      f32x4 v[U][2];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int u = u0 + THREADS * k;
        v[k][0] = v[k][1] = (f32x4){0.f, 0.f, 0.f, 0.f};  // (the last step of the last frame reads up to 31 values, times zero, past its samples)
        if (u >= units) continue;
        // (quotients below 2^20 of whole numbers: half a unit away from the next one, rounding does not matter)
        const int row = (int)(((float)u + 0.5f) * inv_row), col = N * (u - row * per_row);
        const int later = row >= first ? 1 + (int)(((float)(row - first) + 0.5f) * inv_seg) : 0;
        const int sigma = row >= first ? row - first - (later - 1) * seg : tm.t0 + row;
        const int s = sigma * hop + base + col;
        const float* __restrict__ xb = x0 + (long long)later * g.L;
        if (s >= 0 && s <= L - N) {
          v[k][0] = *reinterpret_cast<const f32x4_u*>(xb + s);
          if constexpr (OCTETS) v[k][1] = *reinterpret_cast<const f32x4_u*>(xb + s + 4);
        } else {
          v[k][0] = four(xb, s);
          if constexpr (OCTETS) v[k][1] = four(xb, s + 4);
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int u = u0 + THREADS * k;
        if (u >= units + 32 / N) continue;
        const Planes b = planes(v[k]);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
          unsigned short* to = S + l * plane + place(N * u);
          if constexpr (OCTETS) *reinterpret_cast<u32x4*>(to) = b.p[l];
          else *reinterpret_cast<uint2*>(to) = make_uint2(b.p[l][0], b.p[l][1]);
        }
      }
    }
    __syncthreads();
    for (int s = wk; s < n_step; s += WK) step(steps[s], 32 * s, s + WK < n_step ? s + WK : s);
  }
  {
    if constexpr (WK == 1) {
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[fb][b] = sum[fb][b] * (1.f / (1 << SCALE));
    } else {
      // the waves' sums, through LDS: wave k takes frame block k
      f32x4* const part = reinterpret_cast<f32x4*>(S) + lane;  // [wave][frame block][row block][64 lanes]
      __syncthreads();
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int b = 0; b < RB; ++b) part[((wave * FB + fb) * RB + b) * 64] = sum[fb][b];
      __syncthreads();
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        acc[0][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (wave < FB)
          for (int k = 0; k < WK; ++k) acc[0][b] += part[((k * FB + wave) * RB + b) * 64];
        acc[0][b] *= 1.f / (1 << SCALE);
      }
    }
  }
  bool valid[EB];  // this wave's frames
#pragma unroll
  for (int fb = 0; fb < EB; ++fb) valid[fb] = wave * (16 * EB) + fb * 16 + n < m_valid && (WK == 1 || wave < FB);
  auto finite_sums = [&](int fb, int rb, int u) { return finite(acc[fb][rb][2 * u]) && finite(acc[fb][rb][2 * u + 1]); };
  // `taken`: a bin whose taps meet a sample that is not finite, bit 2 (RB fb + rb) + u
  unsigned taken = 0;
  if (__builtin_expect(*flag, 0)) {  // (out of the way of the others' instructions: 41.05 -> 40.55 us of 16 x 220,500 samples, 84 bins)
    // the tile's samples in units of four, row by row
    const int per_row = width / 4, units = rows_used * per_row;
    auto unit = [&](int u) {
      const int row = u / per_row, col = 4 * (u - row * per_row);
      long long b;
      int sigma;
      tm.decode(row, b, sigma);
      return four(g.x + b * g.L, sigma * hop + item.base - g.pad + col);
    };
    int* const count = reinterpret_cast<int*>(S);
    int2* const list = reinterpret_cast<int2*>(S) + 1;  // place in the tile, value
    unsigned short* const order = S + 4 + 4 * 4 * THREADS;
    __syncthreads();
    if (tid < 2) count[tid] = 0;
    __syncthreads();
    int mine = 0;
#pragma unroll 1
    for (int u = tid; u < units; u += THREADS) {
      const f32x4 v = unit(u);
      for (int e = 0; e < 4; ++e) mine += tame<SCALE>(v[e]) ? 0 : 1;
    }
    atomicAdd(count + 1, mine);
    __syncthreads();
    const bool dense = count[1] > units / 16;
    auto add = [&](int fb, int rb, int u, int tap, const int4& own, float v) {
      const float2 wt = P.taps[own.z + tap - own.x];
      acc[fb][rb][2 * u] += wt.x * v;
      acc[fb][rb][2 * u + 1] += wt.y * v;
      taken |= (finite(v) ? 0u : 1u) << (2 * (RB * fb + rb) + u);
    };
    // few of them: listed a thousand samples at a time, each for the frames it meets
#pragma unroll 1
    for (int u0 = 0; u0 < units && !dense; u0 += THREADS) {
      __syncthreads();
      if (tid == 0) *count = 0;
      __syncthreads();
      if (u0 + tid < units) {
        const f32x4 v = unit(u0 + tid);
        for (int e = 0; e < 4; ++e) {
          const float value = v[e];
          if (!tame<SCALE>(value)) list[atomicAdd(count, 1)] = make_int2(4 * (u0 + tid) + e, __builtin_bit_cast(int, value));
        }
      }
      __syncthreads();
      const int m = *count;
      // (the order of the entries is the waves' chance: by their places, so that every call adds the products in the same order)
#pragma unroll 1
      for (int i = tid; i < m; i += THREADS) {
        int before = 0;
#pragma unroll 1
        for (int j = 0; j < m; ++j) before += list[j].x < list[i].x ? 1 : 0;
        order[before] = (unsigned short)i;
      }
      __syncthreads();
#pragma unroll 1
      for (int i = 0; i < m; ++i) {
        const int2 bad = list[order[i]];
#pragma unroll
        for (int fb = 0; fb < EB; ++fb) {
          const int fi = wave * (16 * EB) + fb * 16 + n, at = bad.x - (valid[fb] ? tm.frame_row(fi) : 0) * width, tap = at + item.base;
          if (!valid[fb] || at < 0 || at >= item.jspan * width) continue;
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int k = 8 * rb + 2 * q + u;
              const int4 own = P.support[item.bin0 + (k < item.n_bins ? k : 0)];
              if (k < item.n_bins && tap >= own.x && tap < own.y) add(fb, rb, u, tap, own, __builtin_bit_cast(float, bad.y));
            }
        }
      }
    }
    // one in 64 or more: every bin looks for them, until it is NaN
#pragma unroll 1
    for (int bit = 0; bit < 2 * RB * EB && dense; ++bit) {
      const int k = 8 * ((bit >> 1) % RB) + 2 * q + (bit & 1), fi = (wave * EB + (bit >> 1) / RB) * 16 + n;
      if (fi >= m_valid || k >= item.n_bins || (WK > 1 && wave >= FB)) continue;
      const long long f = f0 + fi, b = f / g.T;
      const float* __restrict__ xw = g.x + b * g.L;
      const int s0 = (int)(f - b * g.T) * hop - g.pad;
      const int4 own = P.support[item.bin0 + k];
      float re = 0.f, im = 0.f, part_re = 0.f, part_im = 0.f;  // (sums of 16 products, of 256, of all)
      bool met = false, wild = false;
#pragma unroll 1
      for (int tap = own.x; tap < own.y && !(part_re != part_re && part_im != part_im); tap += 16) {
        if ((tap - own.x) % 256 == 0) {
          re += part_re;
          im += part_im;
          part_re = part_im = 0.f;
        }
        f32x4 v[4];
        bool any = false;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (e % 4 == 0) v[e / 4] = four(xw, s0 + tap + e);
          any = any || !tame<SCALE>(v[e / 4][e % 4]);
        }
        if (!any) continue;
        float sum_re = 0.f, sum_im = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (tap + e >= own.y || tame<SCALE>(v[e / 4][e % 4])) continue;
          const float2 wt = P.taps[own.z + tap + e - own.x];
          sum_re += wt.x * v[e / 4][e % 4];
          sum_im += wt.y * v[e / 4][e % 4];
          met = true;
          wild = wild || !finite(v[e / 4][e % 4]);
        }
        part_re += sum_re;
        part_im += sum_im;
      }
      re += part_re;
      im += part_im;
#pragma unroll
      for (int i = 0; i < 2 * RB * EB; ++i) {
        if (i != bit || !met) continue;
        acc[(i >> 1) / RB][(i >> 1) % RB][2 * (i & 1)] += re;
        acc[(i >> 1) / RB][(i >> 1) % RB][2 * (i & 1) + 1] += im;
        taken |= (wild ? 1u : 0u) << i;
      }
    }
  }

  // lane (q, n), registers 0 .. 3 of row block b: (Re, Im) of bins 8 b + 2 q and + 1, frame n of the wave's frame block
  unsigned odd = 0;
#pragma unroll
  for (int fb = 0; fb < EB; ++fb) {
    if (!valid[fb]) continue;
    const long long f = f0 + wave * (16 * EB) + fb * 16 + n, b = f / g.T;
    float* __restrict__ op = P.out + b * P.out_wave_stride + (f - b * g.T);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = 8 * rb + 2 * q + u;
        if (k >= item.n_bins) continue;
        store_bin(P.fmt, g.T, op, item.bin0 + k, acc[fb][rb][2 * u], acc[fb][rb][2 * u + 1]);
        odd |= (finite_sums(fb, rb, u) ? 0u : 1u) << (2 * (RB * fb + rb) + u);
      }
  }
  // Sums that are not finite though all their samples are: the bfloat16 of samples next to the largest float32 overflow together.  Tap by tap.
  odd &= ~taken;
#pragma unroll 1
  while (__builtin_expect(odd, 0)) {
    const int bit = __builtin_ctz(odd), k = 8 * ((bit >> 1) % RB) + 2 * q + (bit & 1), fi = (wave * EB + (bit >> 1) / RB) * 16 + n;
    odd &= odd - 1;
    const long long f = f0 + fi, b = f / g.T;
    const int t = (int)(f - b * g.T);
    const int4 own = P.support[item.bin0 + k];  // first tap, last tap + 1, where its taps are
    const float* __restrict__ xw = g.x + b * g.L;
    float re = 0.f, im = 0.f;
#pragma unroll 1
    for (int tap = own.x; tap < own.y; ++tap) {
      const float v = xw[reflect_clamped(t * hop - g.pad + tap, L)];
      const float2 wt = P.taps[own.z + tap - own.x];
      re += wt.x * v;
      im += wt.y * v;
    }
    store_bin(P.fmt, g.T, P.out + b * P.out_wave_stride + t, item.bin0 + k, re, im);
  }
}

}  // namespace
}  // namespace nna
