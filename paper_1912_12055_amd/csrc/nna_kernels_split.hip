// The three contractions of the trainable layers on the bfloat16 matrix pipe, at float32 precision.
//
//   forward            C[r, f]  = sum_n W[r, n] xp[f hop + n], then the output format or (backward pass) its derivative
//   bank gradient      gW[r, n] = sum_f G[r, f] xp[f hop + n]
//   waveform gradient  D[f, n]  = sum_r G[r, f] W[r, n], added onto the sample each (frame, tap) pair reads
//
// The kernels are free numbers, so none of the symmetries of the fixed banks is left: these are plain products, bound by the
// matrix pipe.  A float32 a is exactly a0 + a1 + a2, three bfloat16 (each the rounding of what the ones before leave: 8 bits of
// the 24 and a sign at a time, and the full exponent range), and
//     a b = a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0) + terms below 2^-26 |a b|,
// six products whose terms are exact in float32, summed by v_mfma_f32_32x32x16_bf16 into float32 accumulators: sixteen times the
// rate of the float32 instruction for six times the work, and fewer roundings (six per sixteen terms; the float32 instruction
// rounds every two).  Exact holds for magnitudes from 2^-110 to the largest bfloat16, 3.39e38: a smaller one loses low bits (its third
// part falls below the smallest bfloat16), a larger one rounds to infinity.  A sample or weight that is not finite makes everything
// it meets NaN.
//
// A workgroup computes 128 rows x 128 columns, a wave all the rows x 32 columns of its own.  The rows' operand is staged through
// LDS, split on the way in, every value once (two buffers, one barrier per 32 contraction indices); the columns' operand nobody
// else in the workgroup reads, and it goes from memory to the wave's registers.
//
// What bounds it: the matrix pipe is busy 37 to 42 % and the vector ALUs, which split the operands, 30 to 46 % (16 x 44,217 samples, the
// three kernels, counters); with two waves per SIMD the two overlap in part.  64 x 110,250 samples, n_fft 2,048 (116 GFLOP each, MI355X; float32 instruction before): contraction 1,045 ->
// 650 us, bank gradient 1,000 -> 640 us; 16 x 44,217: bank gradient 146 -> 117 us, waveform gradient 177 -> 95 us.  Errors against
// 64 bits there: output 6.6e-7 -> 4.7e-7, bank gradient 1.29e-6 -> 9.3e-7.
#include "nna_device.h"

#include <algorithm>
#include <type_traits>

namespace nna {
namespace {

typedef f32x4 f32x4_u __attribute__((aligned(4)));

constexpr int SP_T = 128;      // rows and columns of a tile
constexpr int SP_KC = 32;      // contraction indices per chunk
constexpr int SP_PITCH = 20;   // words per row of a staged plane: 32 bfloat16 and a pad (conflict-free 16-byte reads)
constexpr int SP_PLANE = SP_T * SP_PITCH;

// acc[s] += the products of ROWS 32-row blocks of the staged chunk with this wave's columns
template <int ROWS, int N>
__device__ __forceinline__ void multiply(f32x16 (&acc)[N], const unsigned* __restrict__ lds, const Planes (&b)[2], int h, int r32) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int s0 = 0; s0 < ROWS; s0 += 2) {
      constexpr int two = 2;
      bf16x8 a[two][3];
#pragma unroll
      for (int s = 0; s < two; ++s)
        if (s0 + s < ROWS)
#pragma unroll
          for (int l = 0; l < 3; ++l)
            a[s][l] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(lds + l * SP_PLANE + ((s0 + s) * 32 + r32) * SP_PITCH + 8 * ks + 4 * h));
      // small terms first
      constexpr int la[6] = {2, 1, 0, 1, 0, 0}, lb[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
      for (int m = 0; m < 6; ++m)
#pragma unroll
        for (int s = 0; s < two; ++s)
          if (s0 + s < ROWS)
            acc[s0 + s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s][la[m]], __builtin_bit_cast(bf16x8, b[ks].p[lb[m]]), acc[s0 + s], 0, 0, 0);
    }
}

// The pipeline all three share.  fetch_rows(c, i, v): the eight values of this thread's i-th octet (i = 0, 1) of the rows' operand
// in chunk c; fetch_cols(c, v): this lane's sixteen values of the columns' operand, v[ks] its indices 16 ks + 8 h + 0 .. 7;
// fix_cols(v): what is left to do to them once they are there.  row_word(i): LDS word of octet i.
// PAIRED: two chunks per turn of the loop, no copies of the columns' planes (more registers).  OCTETS of rows a thread (half for 64 rows).
template <int ROWS, bool PAIRED, int OCTETS = 2, int N, typename FR, typename FC, typename FX, typename RW>
__device__ __forceinline__ void contract(f32x16 (&acc)[N], unsigned* __restrict__ lds, long long c_begin, long long c_end, int h, int r32,
                                         FR fetch_rows, FC fetch_cols, FX fix_cols, RW row_word) {
#pragma unroll
  for (int s = 0; s < N; ++s)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[s][r] = 0.f;
  f32x4 ra[OCTETS][2], rb[2][2];
  auto request = [&](long long c) {
#pragma unroll
    for (int i = 0; i < OCTETS; ++i) fetch_rows(c, i, ra[i]);
    fetch_cols(c, rb);
  };
  auto stage = [&](int buf, Planes (&b)[2]) {
    fix_cols(rb);
#pragma unroll
    for (int i = 0; i < OCTETS; ++i) {
      const Planes o = split8(ra[i]);
#pragma unroll
      for (int l = 0; l < 3; ++l) *reinterpret_cast<u32x4*>(lds + (buf * 3 + l) * SP_PLANE + row_word(i)) = o.p[l];
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) b[ks] = split8(rb[ks]);
  };
  Planes b0[2], b1[2];
  request(c_begin);
  stage(0, b0);
  request(c_begin + 1 < c_end ? c_begin + 1 : c_begin);
  __syncthreads();
  if constexpr (!PAIRED) {
    for (long long c = c_begin; c < c_end; ++c) {
      const int buf = (int)(c - c_begin) & 1;
      b1[0] = b0[0];
      b1[1] = b0[1];
      stage(buf ^ 1, b0);
      request(c + 2 < c_end ? c + 2 : c_end - 1);
      multiply<ROWS>(acc, lds + buf * 3 * SP_PLANE, b1, h, r32);
      __syncthreads();
    }
    return;
  }
  for (long long c = c_begin; c < c_end; c += 2) {
    // (behind the last chunk: the last one again, staged and never read)
    stage(1, b1);
    request(c + 2 < c_end ? c + 2 : c_end - 1);
    multiply<ROWS>(acc, lds, b0, h, r32);
    __syncthreads();
    if (c + 1 >= c_end) break;
    stage(0, b0);
    request(c + 3 < c_end ? c + 3 : c_end - 1);
    multiply<ROWS>(acc, lds + 3 * SP_PLANE, b1, h, r32);
    __syncthreads();
  }
}

// ---- forward ------------------------------------------------------------------------------------
// MODE: ST_MODE_STFT, ST_MODE_CPLX or ST_MODE_GRAD (power format), as in the float32 kernel, whose accumulator layout and epilogues
// these are.
// ROWS: 32-row blocks of a tile, four or (short batches) two.
template <int MODE, int ROWS>
__global__ __launch_bounds__(256, 2) void split_forward_kernel(const StftParams P, const float* __restrict__ wrm, int kp, int K) {
  __shared__ __attribute__((aligned(16))) unsigned lds[2 * 3 * SP_PLANE];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5, r32 = lane & 31;
  const FrameGeom& g = P.g;
  // the row tiles of a frame tile are neighbours on one XCD: they share its samples in the L2
  const int n_rt = P.n_rt * (4 / ROWS);
  const long long local = blockIdx.x >> 3, ft = (blockIdx.x & 7) * ((P.n_ft + 7) >> 3) + local / n_rt;
  const int rt = (int)(local % n_rt);
  if (ft >= P.n_ft) return;
  const long long f_lane = ft * SP_T + wave * 32 + r32;
  const bool valid = f_lane < g.n_frames;
  const long long f = valid ? f_lane : g.n_frames - 1, b_lane = f / g.T;
  const int t_lane = (int)(f - b_lane * g.T), L = (int)g.L;
  const float* __restrict__ xb = g.x + b_lane * g.L;
  const int pos = t_lane * g.hop - g.pad;
  const int k_end = (K + SP_KC - 1) / SP_KC * SP_KC;
  const bool edge = __builtin_amdgcn_ballot_w64(pos < 0 || pos + k_end > L) != 0;
  unsigned rev = 0;
  const float* __restrict__ wp = wrm + ((long long)rt * (32 * ROWS) + (tid >> 2)) * kp + 8 * (tid & 3);
  f32x16 acc[ROWS];
  contract<ROWS, true, ROWS / 2>(
      acc, lds, 0, k_end / SP_KC, h, r32,
      [&](long long c, int i, f32x4 (&v)[2]) {
        const float* p = wp + (long long)(64 * i) * kp + c * SP_KC;
        v[0] = *reinterpret_cast<const f32x4*>(p);
        v[1] = *reinterpret_cast<const f32x4*>(p + 4);
      },
      [&](long long c, f32x4 (&v)[2][2]) {
        const int s0 = pos + (int)c * SP_KC + 8 * h;
        if (!edge) {
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u >> 1][u & 1] = *reinterpret_cast<const f32x4_u*>(xb + s0 + 16 * (u >> 1) + 4 * (u & 1));
        } else {
          // four samples on one side of either end are a stored run, read backwards behind an end
          rev = 0;
          bool gen = false;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int s = s0 + 16 * (u >> 1) + 4 * (u & 1);
            const int src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
            rev |= (src != s ? 1u : 0u) << u;
            gen |= (unsigned)src > (unsigned)(L - 4);
            v[u >> 1][u & 1] = *reinterpret_cast<const f32x4_u*>(xb + (src < 0 ? 0 : src > L - 4 ? L - 4 : src));
          }
          if (__builtin_amdgcn_ballot_w64(gen) != 0) {  // runs that straddle an end, or reach past the taps: sample by sample
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int s = s0 + 16 * (u >> 1) + 4 * (u & 1);
              const int src = s < 0 ? -s - 3 : s > L - 4 ? 2 * (L - 1) - s - 3 : s;
              if ((unsigned)src > (unsigned)(L - 4)) {
                rev &= ~(1u << u);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[u >> 1][u & 1][e] = xb[reflect_clamped(s + e, L)];
              }
            }
          }
        }
      },
      [&](f32x4 (&v)[2][2]) {
        if (!edge) return;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const f32x4 q = v[u >> 1][u & 1];
          const bool r = (rev >> u) & 1u;
          v[u >> 1][u & 1] = (f32x4){r ? q.w : q.x, r ? q.z : q.y, r ? q.y : q.z, r ? q.x : q.w};
        }
      },
      [&](int i) { return ((tid >> 2) + 64 * i) * SP_PITCH + 4 * (tid & 3); });
  if (!valid) return;
  const int slot_base = rt * (16 * ROWS);
  if constexpr (MODE == ST_MODE_GRAD) {
    const float* __restrict__ gp = P.gout + (b_lane * P.out_bins) * g.T + t_lane;
    float* __restrict__ Gp = P.gbuf + (f >> 5) * ((long long)P.n_rt * ST_ROWS * 32) + (f & 31);
    float* __restrict__ pp = P.pout ? P.pout + (b_lane * P.out_bins) * g.T + t_lane : nullptr;
    stft_grad_tile<NNA_OUT_POWER>(acc, gp, g.T, Gp, 32, slot_base, h, P.n_half, P.packed, pp);
  } else {
    float* __restrict__ op = P.out + (b_lane * P.out_bins) * g.T + t_lane;
    if (MODE == ST_MODE_STFT && P.keep) {
      float* __restrict__ Kp = P.keep + (f >> 5) * ((long long)P.n_rt * ST_ROWS * 32) + (f & 31);
#pragma unroll
      for (int rb = 0; rb < ROWS; ++rb)
#pragma unroll
        for (int u = 0; u < 16; ++u) Kp[(2 * (slot_base + 2 * h + rb * 16 + 4 * (u >> 2) + ((u >> 1) & 1)) + (u & 1)) * 32] = acc[rb][u];
    }
    if constexpr (MODE == ST_MODE_CPLX) {
      if (P.fmt == NNA_OUT_COMPLEX)
        stft_store_tile_complex<NNA_OUT_COMPLEX>(acc, op, g.T, slot_base, h, P.n_half, P.packed);
      else
        stft_store_tile_complex<NNA_OUT_PHASE>(acc, op, g.T, slot_base, h, P.n_half, P.packed);
    } else if (P.fmt == NNA_OUT_MAGNITUDE) {
      stft_store_tile<NNA_OUT_MAGNITUDE>(acc, op, g.T, slot_base, h, P.n_half, P.packed);
    } else if (P.fmt == NNA_OUT_POWER) {
      stft_store_tile<NNA_OUT_POWER>(acc, op, g.T, slot_base, h, P.n_half, P.packed);
    } else {
      stft_store_tile<NNA_OUT_LOG>(acc, op, g.T, slot_base, h, P.n_half, P.packed);
    }
  }
}

// ---- bank gradient ------------------------------------------------------------------------------
// SPARSE: the output tiles of P.tiles only, each with its count of 32-row blocks that hold taps.
template <bool SPARSE>
__device__ __forceinline__ void bank_tile(const BwParams& P, long long bid, unsigned* __restrict__ lds) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5, r32 = lane & 31;
  const FrameGeom& g = P.g;
  const int n_nt = P.kp / BW_NT, n_mt = P.rows_pad / BW_MT;
  const long long tiles = SPARSE ? P.n_tiles : (long long)n_mt * n_nt;
  const long long split = bid / tiles;
  int tile = (int)(bid - split * tiles);
  long long m0;
  int n0, alive_rt = 4;
  if constexpr (SPARSE) {
    // the list is ordered heaviest tile first; neighbours in it go to different dies, which balances them
    const int2 t = P.tiles[tile];
    m0 = (long long)(t.x & 0xffff) * BW_MT;
    n0 = t.y * BW_NT;
    alive_rt = t.x >> 16;
  } else {
    // Workgroup ids are dealt round-robin to the 8 dies, each with an L2 of its own.  Give every die a contiguous
    // run of tiles in row-major order: it then reads only its own rows of G (the large operand).
    if (tiles % 8 == 0) tile = (tile & 7) * (int)(tiles / 8) + (tile >> 3);
    m0 = (long long)(tile / n_nt) * BW_MT;
    n0 = (tile % n_nt) * BW_NT;
  }
  const long long n_chunks = P.gpitch / SP_KC;
  const long long c_begin = split * P.chunks_per_split;
  const long long c_end = c_begin + P.chunks_per_split < n_chunks ? c_begin + P.chunks_per_split : n_chunks;
  if (c_begin >= c_end) return;
  const int tap = n0 + wave * 32 + r32, L = (int)g.L;
  const float* __restrict__ ap = P.gbuf + (m0 + (tid >> 2)) * 32 + 8 * (tid & 3);
  const long long blk = (long long)P.rows_pad * 32;
  // (waveform, frame in it) of the chunk last asked for: chunks are asked for in order, the last one again at the end
  long long at = c_begin, nfb = c_begin * SP_KC / g.T;
  int nft = (int)(c_begin * SP_KC - nfb * g.T);
  const unsigned x_lane = 8 * h * g.hop + wave * 32 + r32;
  f32x16 acc[4];
  auto sweep = [&](auto alive_tag) {
    contract<decltype(alive_tag)::value, !SPARSE>(
        acc, lds, c_begin, c_end, h, r32,
        [&](long long c, int i, f32x4 (&v)[2]) {
          const float* p = ap + c * blk + 64 * 32 * i;  // (row blocks without taps hold whatever G does: staged, not multiplied)
          v[0] = *reinterpret_cast<const f32x4*>(p);
          v[1] = *reinterpret_cast<const f32x4*>(p + 4);
        },
        [&](long long c, f32x4 (&v)[2][2]) {
          if (c != at) {
            at = c;
            nft += SP_KC;
            while (nft >= g.T) {
              nft -= g.T;
              ++nfb;
            }
          }
          // Almost every chunk lies inside one waveform and clear of its mirrored ends (one test for the whole workgroup):
          // a base every lane shares plus a lane offset that never changes.
          const long long lo = (long long)nft * g.hop + n0 - g.pad;
          if (nft + SP_KC <= g.T && nfb < g.B && lo >= 0 && lo + (long long)(SP_KC - 1) * g.hop + BW_NT <= g.L) {
            const float* base = g.x + nfb * g.L + lo;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const float* bi = base + (long long)(16 * (i >> 3) + (i & 7)) * g.hop;  // uniform
              v[i >> 3][(i >> 2) & 1][i & 3] = bi[x_lane];
            }
            return;
          }
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            int t = nft + 16 * (i >> 3) + 8 * h + (i & 7);
            long long b = nfb;
            while (t >= g.T) {
              t -= g.T;
              ++b;
            }
            b = b < g.B ? b : g.B - 1;  // frames past the last one: their G is zero, any sample serves
            int j = t * g.hop + tap - g.pad;
            j = j < 0 ? -j : j;
            j = j >= L ? 2 * (L - 1) - j : j;  // mirror padding folded back
            j = j < 0 ? 0 : (j >= L ? L - 1 : j);  // taps of the padding columns past K: never stored
            v[i >> 3][(i >> 2) & 1][i & 3] = g.x[b * g.L + j];
          }
        },
        [](f32x4 (&)[2][2]) {}, [&](int i) { return ((tid >> 2) + 64 * i) * SP_PITCH + 4 * (tid & 3); });
  };
  if constexpr (SPARSE) {
    switch (alive_rt) {
      case 1: sweep(std::integral_constant<int, 1>{}); break;
      case 2: sweep(std::integral_constant<int, 2>{}); break;
      case 3: sweep(std::integral_constant<int, 3>{}); break;
      default: sweep(std::integral_constant<int, 4>{}); break;
    }
  } else {
    sweep(std::integral_constant<int, 4>{});
  }
  // accumulator register r of lane (h, r32) of block s is output row m0 + 32 s + 8 (r/4) + 4 h + r%4, column `tap`
  if (tap >= P.K) return;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s >= alive_rt) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int pr = (int)m0 + s * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
      if ((pr >> 1) < P.n_half && (!SPARSE || (tap >= P.row_lo[pr] && tap < P.row_hi[pr]))) {
        const int row = P.packed ? (pr == 0 ? 0 : pr == 1 ? 2 * P.n_half : pr) : pr;  // row of the logical [2 bins][K] bank
        unsafeAtomicAdd(P.gw + (long long)row * P.K + tap, acc[s][r]);
      }
    }
  }
}

// ---- waveform gradient --------------------------------------------------------------------------
__device__ __forceinline__ void wave_tile(const BwParams& P, long long bid, unsigned* __restrict__ lds) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5, r32 = lane & 31;
  const FrameGeom& g = P.g;
  // the tap tiles of one frame tile are neighbours: they share its G columns in the L2
  const int n_nt = P.kp / BW_NT;
  const long long tiles = P.gpitch / BW_MT * n_nt, split = bid / tiles, tile = bid - split * tiles;
  const long long m0 = tile / n_nt * BW_MT;
  const int n0 = (int)(tile % n_nt) * BW_NT;
  const long long c_all = (2 * P.n_half + SP_KC - 1) / SP_KC;  // (the padding rows of G and W are zero)
  const long long c_begin = split * P.chunks_per_split, c_end = c_begin + P.chunks_per_split < c_all ? c_begin + P.chunks_per_split : c_all;
  if (c_begin >= c_end) return;
  // octet i of this thread: frame m0 + tid % 128, bank rows 8 (tid / 128 + 2 i) + 0 .. 7 of the chunk
  const int fr = tid & 127, o0 = tid >> 7;
  const float* __restrict__ ap = P.gbuf + ((m0 + fr) >> 5) * ((long long)P.rows_pad * 32) + (fr & 31) + 8 * o0 * 32;
  const int tap = n0 + wave * 32 + r32;
  const unsigned w_lane = 8 * h * P.kp + tap;
  f32x16 acc[4];
  contract<4, true>(
      acc, lds, c_begin, c_end, h, r32,
      [&](long long c, int i, f32x4 (&v)[2]) {
        const float* p = ap + (c * SP_KC + 16 * i) * 32;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e >> 2][e & 3] = p[e * 32];
      },
      [&](long long c, f32x4 (&v)[2][2]) {
        const float* p = P.wrm + c * SP_KC * P.kp;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float* pi = p + (long long)(16 * (i >> 3) + (i & 7)) * P.kp;  // uniform
          v[i >> 3][(i >> 2) & 1][i & 3] = pi[w_lane];
        }
      },
      [](f32x4 (&)[2][2]) {}, [&](int i) { return fr * SP_PITCH + 4 * (o0 + 2 * i); });
  // accumulator register r of lane (h, r32) of block s is frame m0 + 32 s + 8 (r/4) + 4 h + r%4, column `tap`
  if (tap >= P.K) return;
  const int L = (int)g.L;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      long long f = m0 + s * 32 + 8 * q + 4 * h, b = f / g.T;
      int t = (int)(f - b * g.T);
#pragma unroll
      for (int i = 0; i < 4; ++i, ++f) {
        if (f < g.n_frames) {
          int j = t * g.hop + tap - g.pad;
          j = j < 0 ? -j : (j >= L ? 2 * (L - 1) - j : j);  // mirror padding folded back
          unsafeAtomicAdd(P.gx + b * g.L + j, acc[s][4 * q + i]);
        }
        if (++t == g.T) {
          t = 0;
          ++b;
        }
      }
    }
}

template <bool SPARSE>
__global__ __launch_bounds__(256, 2) void split_bank_kernel(const BwParams P) {
  __shared__ __attribute__((aligned(16))) unsigned lds[2 * 3 * SP_PLANE];
  bank_tile<SPARSE>(P, blockIdx.x, lds);
}

__global__ __launch_bounds__(256, 2) void split_wave_kernel(const BwParams P) {
  __shared__ __attribute__((aligned(16))) unsigned lds[2 * 3 * SP_PLANE];
  wave_tile(P, blockIdx.x, lds);
}

// Both gradients of a step in one launch: neither's tiles fill a short batch's chip.  The backward call, power, against two launches: 16 x
// 44,217 samples, n_fft 2,048, 300 -> 293 us; 2 x 30,000 180 -> 163; n_fft 512, 20 x 60,000 166 -> 153; n_fft 4,096, 4 x 30,000 358 -> 347.  The
// pieces are those of the launches by themselves: uncut where all tiles fill the chip once, a bank of few tiles is a few workgroups' chain over
// all frames (n_fft 512, 30 x 60,000: 184 -> 791 us) and its sums are up to five times further from 64 bits.
__global__ __launch_bounds__(256, 2) void split_both_kernel(const BwParams bank, const BwParams wave, unsigned n_wave) {
  __shared__ __attribute__((aligned(16))) unsigned lds[2 * 3 * SP_PLANE];
  if (blockIdx.x < n_wave)
    wave_tile(wave, blockIdx.x, lds);
  else
    bank_tile<false>(bank, blockIdx.x - n_wave, lds);
}

}  // namespace

hipError_t launch_split_forward(StftParams P, int mode, const float* wrm, int kp, int K, hipStream_t stream) {
  clear_stale_error();
  P.n_ft = (P.g.n_frames + SP_T - 1) / SP_T;
  const long long blocks = (P.n_ft + 7) / 8 * 8 * P.n_rt;
  if (blocks <= 0 || 2 * blocks > 0x7fffffffLL || kp < (K + SP_KC - 1) / SP_KC * SP_KC) return hipErrorInvalidValue;
  if (mode == ST_MODE_GRAD && P.fmt != NNA_OUT_POWER) return hipErrorInvalidValue;
  auto run = [&](auto kernel, long long n) { hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(256), 0, stream, P, wrm, kp, K); };
  // Few tiles: half the rows each.  A whole step, n_fft 2,048, 48 tiles: 340 -> 311 us; n_fft 400, 96: 146 -> 137; Mel, n_fft 1,024, 120: 282 ->
  // 267; n_fft 4,096, 128: 811 -> 796; n_fft 2,048, 176: 345 -> 354, 496: 830 -> 857.  The row tiles of a frame tile share an XCD, which holds 64
  // workgroups: no more than that of them (n_fft 8,192, one and two frame tiles: 914 -> 1,046, 1,142 -> 1,266).
  const bool half = P.n_ft * P.n_rt < 160 && 2 * ((P.n_ft + 7) / 8) * P.n_rt <= 64;
  if (mode == ST_MODE_GRAD) run(split_forward_kernel<ST_MODE_GRAD, 4>, blocks);
  else if (mode == ST_MODE_CPLX) half ? run(split_forward_kernel<ST_MODE_CPLX, 2>, 2 * blocks) : run(split_forward_kernel<ST_MODE_CPLX, 4>, blocks);
  else half ? run(split_forward_kernel<ST_MODE_STFT, 2>, 2 * blocks) : run(split_forward_kernel<ST_MODE_STFT, 4>, blocks);
  return hipGetLastError();
}

hipError_t launch_split_bank(const BwParams& p, hipStream_t stream) {
  clear_stale_error();
  const long long tiles = p.tiles ? p.n_tiles : (long long)(p.rows_pad / BW_MT) * (p.kp / BW_NT);
  const long long blocks = tiles * p.n_split;
  if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (p.tiles)
    hipLaunchKernelGGL(split_bank_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL(split_bank_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

// blocks of a launch of the waveform gradient; sets p.chunks_per_split
static long long shape_wave(BwParams& p) {
  // A short batch's contraction over the bank's rows is halved, or cut into pieces of sixteen chunks until there is a workgroup per compute
  // unit.  A whole step, n_fft 2,048, 176 tiles: 449 us whole, 427 halved, 456 in three (every piece adds onto the waveform by
  // itself); 48 tiles 311, 298, 290, 287 in four; 352 tiles the same either way; 496 tiles 830, 840; n_fft 512, sixteen chunks, 376 tiles: 249, 270.
  const long long tiles = p.gpitch / BW_MT * (p.kp / BW_NT), chunks = (2 * p.n_half + SP_KC - 1) / SP_KC;
  const long long split = tiles > 0 && tiles < 256 && chunks >= 32 ? std::min((256 + tiles - 1) / tiles, chunks / 16) : 1;
  p.chunks_per_split = std::max(1LL, (chunks + split - 1) / split);
  return tiles * ((chunks + p.chunks_per_split - 1) / p.chunks_per_split);
}

hipError_t launch_split_wave(BwParams p, hipStream_t stream) {
  clear_stale_error();
  const long long blocks = shape_wave(p);
  if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(split_wave_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_split_both(const BwParams& p, hipStream_t stream) {
  clear_stale_error();
  BwParams wave = p;
  const long long n_wave = shape_wave(wave), n_bank = (long long)(p.rows_pad / BW_MT) * (p.kp / BW_NT) * p.n_split;
  if (p.tiles || n_wave <= 0 || n_bank <= 0 || n_wave + n_bank > 0x7fffffffLL) return hipErrorInvalidValue;
  if (n_wave + n_bank > 1536) {  // each fills the chip by itself (1,920 workgroups: the step 1,523 us in two launches, 1,531 in one)
    const hipError_t e = launch_split_bank(p, stream);
    return e == hipSuccess ? launch_split_wave(p, stream) : e;
  }
  hipLaunchKernelGGL(split_both_kernel, dim3((unsigned)(n_wave + n_bank)), dim3(256), 0, stream, p, wave, (unsigned)n_wave);
  return hipGetLastError();
}

}  // namespace nna
