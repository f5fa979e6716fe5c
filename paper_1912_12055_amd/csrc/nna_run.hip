// Running a plan: shape checks, launch parameters and the transform calls of the C ABI, the per-device
// set-up, and the library's static workspace with the entry point that uses it.
#include "nna_host.h"

// Workspace of nna_cqt2010v2_static: the downsampled waveforms of two consecutive octaves live here instead
// of in caller memory.  Every device the library's code is loaded on holds its own copy of the array, at its
// own address; in host code the name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[NNA_STATIC_SCRATCH_BYTES];

namespace nna {
namespace host {

// ---- device helpers -----------------------------------------------------------------
// Per-device set-up, done once on every device a plan is built for (that device current): the kernels'
// dynamic-LDS attribute, and the address of this device's copy of `scratch`.
std::mutex g_init_mutex;
std::vector<char> g_init_done;
std::vector<void*> g_scratch_ptr;
hipError_t ensure_kernels_init(int device) {
  std::lock_guard<std::mutex> lock(g_init_mutex);
  if ((int)g_init_done.size() <= device) {
    g_init_done.resize(device + 1, 0);
    g_scratch_ptr.resize(device + 1, nullptr);
  }
  if (!g_init_done[device]) {
    hipError_t e = nna::kernels_init();
    if (e == hipSuccess) e = nna::cqf_kernels_init();
    if (e == hipSuccess) e = nna::cql_kernels_init();
    if (e == hipSuccess) e = nna::short_kernels_init();
    if (e == hipSuccess) e = nna::fft_kernels_init();
    if (e != hipSuccess) return e;
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    g_init_done[device] = 1;
  }
  return hipSuccess;
}

// this device's `scratch`, or NULL if no plan was ever built for it
void* scratch_of(int device) {
  std::lock_guard<std::mutex> lock(g_init_mutex);
  return device >= 0 && device < (int)g_scratch_ptr.size() ? g_scratch_ptr[device] : nullptr;
}

// frames per waveform, or 0 if the signal is too short
long long frames_of(const nna_plan* p, long long L) {
  if (p->center) {
    if (L <= p->pad) return 0;  // mirror reflection needs pad <= L-1
  } else if (L < p->K) {
    return 0;
  }
  return 1 + (L + 2LL * p->pad - p->K) / p->hop;
}

// Largest frame tile (<= cap) whose LDS rows  M + segments(M,T)*extra  fit in `rows_max`.
int pick_tile_frames(int cap, long long T, int extra, int rows_max) {
  for (int M = cap; M >= 1; --M) {
    const long long nseg = 1 + (M - 1 + T - 1) / T;
    if ((long long)M + nseg * extra <= rows_max) return M;
  }
  return 0;
}

nna_status check_call(const nna_plan* plan, int kind, const float* x, long long B, long long L, float* out,
                      long long* T_out) {
  if (!plan) return fail(NNA_ERR_INVALID_ARG, "plan is NULL");
  if (plan->kind != kind) return fail(NNA_ERR_INVALID_ARG, "plan was built for a different transform");
  if (!x || !out) return fail(NNA_ERR_INVALID_ARG, "x_dev / out_dev is NULL");
  if (plan->device < 0) return fail(NNA_ERR_UNSUPPORTED, "host-only plan (device = -1) cannot run transforms");
  if (B < 1) return fail(NNA_ERR_SHAPE, "B must be >= 1");
  // the framing loader fetches windows of four consecutive stored samples
  if (L < 4) return fail(NNA_ERR_SHAPE, "L must be at least 4 samples");
  const long long T = frames_of(plan, L);
  if (T < 1) return fail(NNA_ERR_SHAPE, plan->center ? "L must exceed the reflection padding (K/2)" : "L is shorter than one window");
  // the kernels index samples of one waveform with 32-bit integers (padded index < L + 2K)
  if (T > 0x7fffffffLL / 4 || L > 0x7fffffffLL - 4LL * plan->K - 64 || B > 0x7fffffffLL || B > (1LL << 40) / T)
    return fail(NNA_ERR_SHAPE, "batch too large");
  *T_out = T;
  return NNA_OK;
}

nna::FrameGeom make_geom(const nna_plan* p, const float* x, long long B, long long L, long long T) {
  nna::FrameGeom g;
  g.x = x;
  g.B = B;
  g.L = L;
  g.T = (int)T;
  g.n_frames = B * T;
  g.hop = p->hop;
  g.pad = p->pad;
  g.vec_ok = (L % 4 == 0) && (p->hop % 4 == 0) && (p->pad % 4 == 0) && ((reinterpret_cast<uintptr_t>(x) & 15) == 0);
  return g;
}

// One launch of the STFT kernel family: T frames of each of the B waveforms (arguments checked by the
// caller).  out_wave_stride / row_offset place a two-stage CQT plan's rows inside a larger output
// (octave of a downsampling plan); 0 / 0 = the plan's own [B, bins, T].
nna_status run_stft_core(const nna_plan* plan, int kind, const float* x, long long B, long long L, long long T,
                         float* out, long long out_wave_stride, int row_offset, void* stream, float* spec_out, float* keep) {
  if (plan->precision == NNA_PREC_F16) {
    const int M = pick_tile_frames(nna::H_FRAMES, T, plan->nj - 1, nna::H_LB_ROWS);
    if (M < 1) return fail(NNA_ERR_UNSUPPORTED, "frame tile does not fit in LDS");
    nna::Stft16Params P;
    std::memset(&P, 0, sizeof(P));
    P.g = make_geom(plan, x, B, L, T);
    P.bank = plan->d_bank16;
    P.bank_s = plan->d_bank16s;
    P.out = out;
    P.n_rt = plan->n_rt16;
    P.n_chunks = plan->hop / nna::H_KC;
    P.nj = plan->nj;
    P.n_half = plan->n_half;
    P.packed = plan->freq_scale ? 0 : 1;
    P.out_bins = plan->stft_bins();
    P.fmt = plan->fmt;
    P.rt_per_block = plan->n_rt16;
    P.tile_frames = M;
    P.n_ft = (P.g.n_frames + M - 1) / M;
    DeviceGuard guard;
    hipError_t e = guard.enter(plan->device);
    if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
    e = nna::launch_stft16(P, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return NNA_OK;
  }
  if (plan->runs_fft() && B * T <= plan->fft_frames && (kind == NNA_KIND_STFT || kind == NNA_KIND_MEL)) {
    nna::FftParams P;
    std::memset(&P, 0, sizeof(P));
    P.g = make_geom(plan, x, B, L, T);
    P.win = plan->d_fft_win;
    P.tw = reinterpret_cast<const float2*>(plan->d_fft_tw);
    P.tw_lane = reinterpret_cast<const float4*>(plan->d_fft_lane);
    P.out = out;
    P.spec = spec_out;
    P.M = plan->K / 2;
    P.fmt = plan->fmt;
    P.n_radix = plan->fft_n_radix;
    std::copy(plan->fft_radix, plan->fft_radix + 16, P.radix);
    int mode = plan->fmt == NNA_OUT_COMPLEX || plan->fmt == NNA_OUT_PHASE ? nna::FFT_MODE_CPLX : nna::FFT_MODE_POWER;
    if (kind == NNA_KIND_MEL) {
      mode = nna::FFT_MODE_MEL;
      P.mel = reinterpret_cast<const int4*>(plan->d_fft_mel);
      P.melw = reinterpret_cast<const float4*>(plan->d_fft_melw);
      P.mel_quads = (int)(plan->h_fft_melw.size() / 4);
      P.n_mels = plan->n_mels;
      P.mel_power = plan->mel_power;
    }
    DeviceGuard guard;
    hipError_t e = guard.enter(plan->device);
    if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
    e = nna::launch_stft_fft(P, mode, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return NNA_OK;
  }
  // The folded kernel addresses the rows of a frame tile as 32-bit byte offsets from the tile's first waveform:
  // the waveforms a tile can span must lie within 2^31 bytes (else the direct kernel runs).
  // (chunks visited in pairs: a tile also holds the mirrored partners' rows, J/2 further on)
  const bool fold_pair = plan->runs_split() && plan->fold_pair;
  const int fold_M = plan->runs_folded() ? pick_tile_frames(ST_FRAMES, T, fold_pair ? plan->nj - 1 : plan->nj / 2 - 1, nna::SF_LDS_ROWS) : 0;
  const bool fold_fits = fold_M >= 1 && (1 + (fold_M - 1 + T - 1) / T) * L <= (1LL << 29);
  // (the Mel launch split by tap parity can write the spectrogram it forms on the way; the once-folded one cannot)
  if (fold_fits && (!spec_out || (kind == NNA_KIND_MEL && plan->runs_split())) && (kind == NNA_KIND_STFT || kind == NNA_KIND_MEL)) {
    const int nj2 = plan->nj / 2;
    const int M = fold_M;
    nna::StftParams P;
    std::memset(&P, 0, sizeof(P));
    P.g = make_geom(plan, x, B, L, T);
    P.bankf = reinterpret_cast<const float4*>(plan->d_bankf);
    P.wn = plan->d_wn;
    P.wmid = plan->wmid;
    P.out = out;
    P.n_rt = plan->n_rt;
    P.n_chunks = plan->n_chunks;
    P.nj = nj2;
    P.n_half = plan->n_half;
    P.packed = 0;
    P.tile_frames = M;
    P.n_ft = (P.g.n_frames + M - 1) / M;
    if (kind == NNA_KIND_MEL) {
      P.out_bins = plan->n_mels;
      P.fmt = plan->mel_power;
      P.melw = reinterpret_cast<const float4*>(plan->d_melwf);
      P.mel_mask = plan->d_mel_maskf;
      P.mel_pass_rt = plan->d_mel_pass_rt;
      P.n_mels = plan->n_mels;
      P.n_pass = plan->n_pass;
      if (plan->runs_split()) {  // 32-bin row tiles below N/4, their own pass table; bin N/4 weighed in at the end
        P.split = 1;
        P.pair = plan->fold_pair ? 1 : 0;
        P.n_rt = plan->n_rt_split;
        P.mel_pass_rt = plan->d_mel_pass_rtf;
        P.wn = plan->d_wq;
        P.mel_wnyq = plan->d_mel_wq;
        P.mel_nyq_any = plan->mel_q_any;
        if (spec_out) {
          P.pout = spec_out;
          P.mel_pass_rt = plan->d_mel_pass_rtf_spec;
        }
      }
    } else {
      P.out_bins = plan->n_half + 1;
      P.fmt = plan->fmt;
      if (plan->runs_split()) {  // the bins below N/4 only; bin N/4 from the workgroups behind the contraction's
        P.split = 1;
        P.pair = plan->fold_pair ? 1 : 0;
        P.n_rt = plan->n_rt_split;
        P.wn = plan->d_wq;
      }
      const long long ft_per_xcd = (P.n_ft + 7) / 8;
      P.main_blocks = 8 * ((ft_per_xcd + 63) / 64) * 64 * ((P.n_rt + nna::ST_RG - 1) / nna::ST_RG);
    }
    DeviceGuard guard;
    hipError_t e = guard.enter(plan->device);
    if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
    e = nna::launch_stft_fold(P, kind == NNA_KIND_MEL ? nna::ST_MODE_MEL : nna::ST_MODE_STFT, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return NNA_OK;
  }
  const bool cplx = kind == NNA_KIND_STFT && (plan->fmt == NNA_OUT_COMPLEX || plan->fmt == NNA_OUT_PHASE);
  int lds_rows = kind == NNA_KIND_CQT1992 && plan->lin_blocks == 6 ? nna::ST_LDS_ROWS_WIDE : ST_LDS_ROWS;
  // complex / phase output with many hop-shifts: the one-workgroup-per-CU build when its 192-row tile holds more than
  // 8/7 of the frames the 160-row tile does
  const bool wide = cplx && pick_tile_frames(ST_FRAMES, T, plan->nj - 1, nna::ST_LDS_ROWS_WIDE) * 7 >
                                pick_tile_frames(ST_FRAMES, T, plan->nj - 1, ST_LDS_ROWS) * 8;
  if (wide) lds_rows = nna::ST_LDS_ROWS_WIDE;
  const int M = pick_tile_frames(ST_FRAMES, T, plan->nj - 1, lds_rows);
  if (M < 1) return fail(NNA_ERR_UNSUPPORTED, "frame tile does not fit in LDS");
  nna::StftParams P;
  std::memset(&P, 0, sizeof(P));
  P.wide = wide ? 1 : 0;
  P.g = make_geom(plan, x, B, L, T);
  P.bank = reinterpret_cast<const float4*>(plan->d_bank);
  P.out = out;
  P.n_rt = plan->n_rt;
  P.n_chunks = plan->n_chunks;
  P.nj = plan->nj;
  P.n_half = plan->n_half;
  P.packed = plan->freq_scale ? 0 : 1;
  P.out_bins = kind == NNA_KIND_MEL ? plan->n_mels : kind == NNA_KIND_CQT1992 ? plan->n_bins : plan->out_rows();
  P.tile_frames = M;
  P.n_ft = (P.g.n_frames + M - 1) / M;
  if (kind == NNA_KIND_MEL) {
    P.fmt = plan->mel_power;
    P.melw = reinterpret_cast<const float4*>(plan->d_melw);
    P.mel_mask = plan->d_mel_mask;
    P.mel_wnyq = plan->d_mel_wnyq;
    P.mel_pass_rt = plan->d_mel_pass_rt;
    P.n_mels = plan->n_mels;
    P.n_pass = plan->n_pass;
    P.mel_nyq_any = plan->mel_nyq_any;
  } else if (kind == NNA_KIND_CQT1992) {
    P.fmt = plan->fmt;
    P.out_wave_stride = out_wave_stride > 0 ? out_wave_stride : (long long)plan->out_rows() * T;
    P.row_offset = row_offset;
    P.melw = reinterpret_cast<const float4*>(plan->d_melw);
    P.mel_mask = plan->d_mel_mask;
    P.mel_wnyq = plan->d_mel_wnyq;
    P.mel_pass_rt = plan->d_mel_pass_rt;
    P.n_mels = 2 * plan->n_bins;
    P.n_pass = plan->n_pass;
    P.lin_blocks = plan->lin_blocks;
  } else {
    P.fmt = plan->fmt;
  }
  DeviceGuard guard;
  hipError_t e = guard.enter(plan->device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  P.pout = spec_out;
  P.keep = keep;
  const int mode = kind == NNA_KIND_MEL       ? (spec_out ? nna::ST_MODE_MELSPEC : nna::ST_MODE_MEL)
                   : kind == NNA_KIND_CQT1992 ? nna::ST_MODE_LIN
                   : (plan->fmt == NNA_OUT_COMPLEX || plan->fmt == NNA_OUT_PHASE) ? nna::ST_MODE_CPLX
                                                                                  : nna::ST_MODE_STFT;
  if (plan->d_wrm && kind == NNA_KIND_MEL && spec_out) {
    // trained filters are dense: the spectrogram by the split contraction, then filterbank x spectrogram as a product of its own
    P.out = spec_out;
    P.out_bins = plan->n_half + 1;
    P.fmt = plan->mel_power == 1 ? NNA_OUT_MAGNITUDE : NNA_OUT_POWER;
    e = nna::launch_split_forward(P, nna::ST_MODE_STFT, plan->d_wrm, plan->kp, plan->K, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    nna::MelBwParams Q;
    std::memset(&Q, 0, sizeof(Q));
    Q.g = spec_out;
    Q.wrm = plan->d_melw_t;
    Q.gP = out;
    Q.B = B;
    Q.T = (int)T;
    Q.F = plan->n_mels;
    Q.n_mels = plan->n_half + 1;
    Q.fp = plan->melt_pitch;
    Q.mels_pad = plan->melt_rows;
    e = nna::launch_mel_bw_spec(Q, reinterpret_cast<hipStream_t>(stream));
  } else if (plan->d_wrm && kind == NNA_KIND_STFT)
    e = nna::launch_split_forward(P, mode, plan->d_wrm, plan->kp, plan->K, reinterpret_cast<hipStream_t>(stream));
  else
    e = nna::launch_stft(P, mode, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return fail_hip(e, "kernel launch");
  return NNA_OK;
}

nna_status run_stft_like(const nna_plan* plan, int kind, const float* x, long long B, long long L, float* out,
                         void* stream) {
  long long T = 0;
  nna_status s = check_call(plan, kind, x, B, L, out, &T);
  if (s != NNA_OK) return s;
  return run_stft_core(plan, kind, x, B, L, T, out, 0, 0, stream);
}

// the kernels folded about their centres (nna_kernels_cqf.hip): M frames per tile
nna_status run_conv_fold(const nna_plan* sub, const float* x, long long B, long long L, long long T, float* out,
                         long long out_wave_stride, int row_offset, int M, void* hip_stream) {
  nna::CqfParams P;
  std::memset(&P, 0, sizeof(P));
  P.g = make_geom(sub, x, B, L, T);
  P.bank = reinterpret_cast<const float4*>(sub->d_bankq);
  P.items = sub->d_qitems;
  P.chunks = sub->d_qchunks;
  P.bins = sub->d_qbins;
  P.out = out;
  P.out_wave_stride = out_wave_stride;
  P.row_offset = row_offset;
  P.n_items = (int)sub->h_qitems.size();
  P.n_chunks = sub->q_n_chunks;
  P.fmt = sub->fmt;
  P.tile_frames = M;
  const int extra = sub->q_max_jspan - 1;
  const long long nseg = 1 + (M - 1 + T - 1) / T;
  P.lds_rows = (int)((M + nseg * extra + 63) / 64 * 64);
  P.centre = sub->K / 2;
  const double turn = std::fmod(sub->Q, 2.0);
  P.rot_c = (float)std::cos(kPi * turn);
  P.rot_s = (float)std::sin(kPi * turn);
  P.n_ft = (P.g.n_frames + M - 1) / M;
  hipError_t e = nna::launch_cqt_fold(P, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return fail_hip(e, "kernel launch");
  return NNA_OK;
}

// The tile of a form of the short kernels, its samples in up to `lds` bytes; false: it holds too few of its frames
bool fit_short(const nna_plan* sub, long long n_frames, long long T, int form, size_t lds, nna::ShortParams& P) {
  P.n_items = (int)sub->h_sitems.size();
  P.form = form;
  int M = 0;
  const bool columns = form >= nna::SHORT_COLUMNS;
  int widths = 0;
  for (const nna::ShortItem& it : sub->h_sitems) widths |= it.width;
  if (columns && widths % 32 != 0) return false;
  P.octets = widths % 8 == 0;
  // by columns: as many at a time as the tile's rows leave room for
  auto tile = [&](int kc) {
    int m = nna::SHORT_FRAMES[form];
    for (const nna::ShortItem& it : sub->h_sitems) {
      const int rows = !columns ? (int)(((long long)(lds - 16) / 6 - 24) * 8 / 9 - 32) / it.width
                       : form == nna::SHORT_COLUMNS ? nna::SHORT_ROWS
                                                    : std::min(nna::SHORT_PASSES * 2048 / kc, (int)((lds - 16) / 6 / (kc + 8)));
      m = std::min(m, pick_tile_frames(m, T, it.jspan - 1, rows));
    }
    P.columns_at_once = kc;
    return m;
  };
  // (the columns past a row's last are read too, and are no more than the hop's)
  auto whole = [&](int kc) {
    return std::all_of(sub->h_sitems.begin(), sub->h_sitems.end(), [&](const nna::ShortItem& it) { return ceil_div(it.width, kc) * kc <= std::max(it.width, sub->hop); });
  };
  if (form <= nna::SHORT_COLUMNS) {
    M = tile(32);
  } else {
    for (int kc = 128; kc >= 32; kc /= 2)
      if (whole(kc) && ((M = tile(kc)) == nna::SHORT_FRAMES[form] || kc == 32)) break;
  }
  if (4 * M < 3 * nna::SHORT_FRAMES[form]) return false;
  const long long nseg = 1 + (M - 1 + T - 1) / T;
  P.plane = nna::SHORT_PLANE_MIN[form];
  for (const nna::ShortItem& it : sub->h_sitems) {
    const long long r = M + nseg * (it.jspan - 1);
    P.plane = std::max(P.plane, columns ? (int)(r * (P.columns_at_once + 8)) : nna::SHORT_PLANE(r * it.width));
  }
  P.tile_frames = M;
  P.n_ft = (n_frames + M - 1) / M;
  return true;
}

void set_short(const nna_plan* sub, nna::ShortParams& P) {
  P.w = reinterpret_cast<const uint4*>(sub->d_sw);
  P.taps = reinterpret_cast<const float2*>(sub->d_staps);
  P.support = sub->d_ssupport;
  P.steps = sub->d_ssteps;
  P.columns = sub->d_scolumns;
  P.items = sub->d_sitems;
}

// The kernels by hop-blocks (nna_kernels_cql.hip).  A tile is 64 frames per 16-frame block of a wave (the registers of a direct
// item hold two such blocks); smaller tiles spread a short batch over the chip.  Two workgroups per CU want 80 KB of LDS each; a
// tile cut below three quarters for that takes one workgroup's 156 KB instead.  False: not a launch for this kernel.  It is one
// where the form that runs otherwise (folded about the centres, or tap by tap) has fewer workgroups than there are CUs (its time over
// the other's, batches of 50 to 13,000 frames, MI355X: 0.02 .. 0.9), or takes 1.25 times the multiply-adds, unfilled tiles and the
// first stage's overlap counted (13,000 to 300,000 frames, theirs over the other's 0.22 .. 0.55: time 0.16 .. 0.46; 0.63 .. 0.67: 0.45
// .. 0.85; 0.73 .. 0.81: 0.38 .. 0.87).  (Beyond the line, 0.84 .. 1.13, the time would still be 0.41 .. 0.74.)
bool shape_lowrank(const nna_plan* sub, long long n_frames, long long T, nna::CqlParams& P) {
  const int n_items = (int)sub->h_litems.size(), n_basis = (int)std::count_if(sub->h_litems.begin(), sub->h_litems.end(), [](const nna::CqlItem& it) { return it.r != 0; });
  P.lds_floats = 0;
  double cost = 0;  // multiply-adds per frame
  for (int direct = 0; direct < 2; ++direct) {
    const int i0 = direct ? n_basis : 0, i1 = direct ? n_items : n_basis;
    nna::CqlPart& part = direct ? P.direct : P.basis;
    part.items = sub->d_litems + i0;
    part.n_items = i1 - i0;
    part.fb = 1;
    if (i0 == i1) continue;
    auto fits = [&](int cap, size_t lds) {
      int M = cap;
      for (int i = i0; i < i1; ++i) {
        const int rows = direct ? nna::CQL_ROWS(cap / 64) : (int)((lds / 4 - 32) / sub->h_litems[i].r);
        M = std::min(M, pick_tile_frames(M, T, sub->h_litems[i].jspan - 1, rows));
      }
      return M;
    };
    int cap = direct ? CQ_FRAMES / 2 : CQ_FRAMES;
    while (cap > 64 && (n_frames + cap - 1) / cap * n_items < 512) cap /= 2;
    int M = fits(cap, nna::CQL_LDS_TWO);
    if (4 * M < 3 * cap) M = fits(cap, nna::CQL_LDS_ONE);
    if (M < 16) return false;
    part.fb = cap / 64;
    part.tile_frames = M;
    part.n_ft = (n_frames + M - 1) / M;
    const long long nseg = 1 + (M - 1 + T - 1) / T;
    // The kernels that stay as they are: by tiles whose waves share their steps (nna_short.h), each reading a quarter of the weights for 64
    // frames, where 128 columns go into LDS at a time or the tiles would hold 64 frames anyway.  22,050 Hz, 84 bins, hop 512, 6,900
    // frames: 58 -> 46 us, 87,000: 438 -> 373; 44.1 kHz, 168 bins, 610,650 frames: 5.81 -> 5.12 ms.  (60 bins of a large batch, tiles of 128
    // frames against these: hop 64 216, 206 us, hop 96 157, 166, hop 160 229, 239.)
    if (direct && (sub->hop % 128 == 0 || part.fb == 1) && !sub->h_sitems.empty() &&
        fit_short(sub, n_frames, T, nna::SHORT_COLUMNS_64, 80 * 1024, P.shorts))
      P.lds_floats = std::max(P.lds_floats, (P.shorts.plane * 6 + 16 + 3) / 4);
    else
      P.shorts.n_items = 0;
    for (int i = i0; i < i1; ++i) {
      const nna::CqlItem& it = sub->h_litems[i];
      if (direct && P.shorts.n_items) break;
      const int rows = (int)(M + nseg * (it.jspan - 1));
      P.lds_floats = std::max(P.lds_floats, direct ? (rows + 31) / 32 * 32 * 2 * (nna::CQL_COLS(part.fb) + 4) : rows * it.r + 32);
      cost += direct ? 0.0 : (16.0 * it.n_ib * sub->hop * rows + 256.0 * (it.n_step + it.s_hi - it.s_lo) * cap) / M;
    }
    if (direct) cost += sub->lr_direct * cap / M;
  }
  const int M0 = pick_tile_frames(CQ_FRAMES, T, (sub->max_jspan - 1) * sub->row_step, CQ_LDS_ROWS_MAX);
  const int Mf = sub->runs_cqfold() ? pick_tile_frames(CQ_FRAMES, T, sub->q_max_jspan - 1, nna::CQF_LDS_ROWS) : 0;
  const bool folds = Mf >= 1 && 2 * Mf >= M0;
  const int M = folds ? Mf : M0;
  if (M < 1 || (n_frames + M - 1) / M * (long long)(folds ? sub->h_qitems.size() : sub->h_items.size()) < 256) return true;
  return cost <= 0.8 * 0.5 * (folds ? sub->exec_flops_cqf : sub->exec_flops) * CQ_FRAMES / M;
}

// The coordinates of a call's hop-blocks in memory: floats of a waveform; zero: no items with a basis
long long coordinates_of(const nna_plan* sub, long long T, int& blocks, int& j0, int& j1) {
  long long floats = 0;
  blocks = j1 = 0;
  j0 = INT_MAX;
  for (const nna::CqlItem& it : sub->h_litems) {
    if (!it.r) continue;
    floats += (long long)it.r * (T + it.jspan - 1);
    blocks += it.n_ib;
    j0 = std::min(j0, it.j0);
    j1 = std::max(j1, it.j0 + it.jspan);
  }
  return floats;
}

// The launch of the first stage by itself: 16-hop-block parts of a tile, the parts that the row blocks of all bases are dealt to.  32
// hop-blocks and twelve row blocks a workgroup fill the chip sooner (16 x 220,500 samples, 84 dense kernels: 33 us; 24 row blocks 41, 64
// hop-blocks 42, both 50); twice as many of both read the weights half as often
void shape_project(long long rows, int blocks, int& nb, int& groups) {
  nb = rows >= 64 * 512 ? 4 : 2;
  const int each = nb == 4 ? 24 : 12;
  groups = (blocks + each - 1) / each;
}

// What a call may use of a workspace, waveforms at a time, up to 256 MiB, what the last-level cache holds (1,770 x 176,400 samples, 168 bins: 64 MB
// 5.12 ms, 128 4.87, 256 4.87, 1 GB 4.76); zero: it does as well without.  Two launches instead of one (time over the one launch's, 624 calls of
// 200 to 400,000 frames, hops of 128 to 1,024, 12 to 36 bins per octave) by what the first stage's multiply-adds come to, done once, its workgroups'
// spare row blocks counted:
// - nothing runs beside the items with a basis: where they get no more (0.52 .. 1.05; more: 0.89 .. 1.10), or bases are of five row blocks and
//   more (0.52 .. 0.96: such tiles leave a compute unit one workgroup);
// - the one launch's items are more than reside at once, what neighbouring tiles share is a sixth of all and a tenth is saved: 0.58 .. 1.04
//   (fewer items 0.74 .. 1.45: the second launch waits for the first; less saved 0.9 .. 1.28);
// - a large batch, the first stage 0.3 of all, a tenth of all more multiply-adds at most and four groups of bins or more that each read every
//   sample: 0.80 .. 1.03 (a smaller stage up to 1.08, fewer groups 0.97 .. 1.14, more multiply-adds 0.75 .. 1.05); at hops of 1,024 and more
//   either of the last two will do: 0.63 .. 0.95 (neither: 1.05, 1.06).
size_t lowrank_workspace(const nna_plan* sub, long long B, long long L, long long T) {
  nna::CqlParams P;
  std::memset(&P, 0, sizeof(P));
  if (!sub->runs_lowrank() || !shape_lowrank(sub, B * T, T, P)) return 0;
  const double M = P.basis.tile_frames, nseg = 1 + (P.basis.tile_frames - 1 + T - 1) / T;
  double first = 0, once = 0, second = 0;  // multiply-adds per frame
  for (const nna::CqlItem& it : sub->h_litems) {
    if (!it.r) continue;
    const double each = 16.0 * it.n_ib * sub->hop;
    first += each * (M + nseg * (it.jspan - 1)) / M;
    once += each * (T + it.jspan - 1.0) / T;
    second += 256.0 * (it.n_step + it.s_hi - it.s_lo) * 64 * P.basis.fb / M;
  }
  int blocks, j0, j1, nb, groups;
  const long long floats = coordinates_of(sub, T, blocks, j0, j1);
  shape_project(B * (T + j1 - j0 - 1), blocks, nb, groups);
  const int slots = groups * (blocks <= 12 * groups ? 12 : 24);
  const double all = first + second + sub->lr_direct, saved = first - once * slots / blocks;
  const int items = P.basis.n_items;
  const bool pays = !P.direct.n_items ? saved >= 0 || blocks >= 5 * items
                    : (first - once >= all / 6 && saved >= all / 10 && P.basis.n_ft * items >= 512) ||
                          (B * T >= 50000 && first >= 0.3 * all &&
                           (sub->hop >= 1024 ? items >= 4 || saved >= -all / 10 : items >= 4 && saved >= -all / 10));
  if (!pays) return 0;
  const long long bytes = 4 * floats;
  constexpr long long most = 256LL << 20;
  return bytes > most ? 0 : (size_t)(bytes * std::min(B, most / bytes));
}

nna_status run_conv_lowrank(const nna_plan* sub, const float* x, long long B, long long L, long long T, float* out,
                            long long out_wave_stride, int row_offset, nna::CqlParams& P, void* hip_stream, void* workspace = nullptr,
                            size_t workspace_bytes = 0) {
  int blocks, j0, j1;
  const long long floats = coordinates_of(sub, T, blocks, j0, j1);
  long long at_once = workspace ? (long long)(workspace_bytes / 4) / floats : 0;
  if (at_once > 0 && at_once < B) {
    // As many waveforms at a time as the workspace holds the coordinates of, in parts of equal size.  A part too short for this kernel's
    // tiles: all of them in one launch, which needs no workspace.
    const long long parts = (B + at_once - 1) / at_once;
    nna::CqlParams Q;
    auto shape = [&](long long n) {
      std::memset(&Q, 0, sizeof(Q));
      return shape_lowrank(sub, n * T, T, Q);
    };
    if (!shape(B / parts) || !shape((B + parts - 1) / parts)) at_once = 0;
    for (long long i = 0; at_once && i < parts; ++i) {
      const long long b0 = B * i / parts, n = B * (i + 1) / parts - b0;
      shape(n);
      const nna_status s = run_conv_lowrank(sub, x + b0 * L, n, L, T, out + b0 * out_wave_stride, out_wave_stride, row_offset, Q, hip_stream, workspace, workspace_bytes);
      if (s != NNA_OK) return s;
    }
    if (at_once) return NNA_OK;
  }
  P.g = make_geom(sub, x, B, L, T);
  P.u = reinterpret_cast<const float4*>(sub->d_lu);
  P.a = reinterpret_cast<const float4*>(sub->d_la);
  P.ub = reinterpret_cast<const uint4*>(sub->d_lub);
  P.ab = reinterpret_cast<const uint4*>(sub->d_lab);
  P.steps = sub->d_lsteps;
  P.support = sub->d_lsupport;
  P.out = out + (long long)row_offset * T;
  P.out_wave_stride = out_wave_stride;
  P.fmt = sub->fmt;
  if (P.shorts.n_items) {
    nna::ShortParams& s = P.shorts;
    s.g = P.g;
    set_short(sub, s);
    s.out = P.out;
    s.out_wave_stride = out_wave_stride;
    s.fmt = sub->fmt;
    P.direct = nna::CqlPart{};
    P.direct.fb = 1;
  }
  if (at_once > 0) {
    P.y = static_cast<float*>(workspace);
    P.y_wave = floats;
    P.y_j0 = j0;
    P.y_rows = (int)T + j1 - j0 - 1;
    P.y_blocks = blocks;
    shape_project(B * P.y_rows, blocks, P.y_nb, P.y_groups);
    // the coordinates' words, and the waves' sums where they keep the workgroup in half a CU's LDS, or all of it
    int words = 0;
    const long long nseg = 1 + (P.basis.tile_frames - 1 + T - 1) / T;
    for (const nna::CqlItem& it : sub->h_litems)
      if (it.r) words = std::max(words, (int)(P.basis.tile_frames + nseg * (it.jspan - 1)) * it.r + 32);
    if (P.shorts.n_items) P.lds_floats = words;
    const int with_sums = (words + 3) / 4 * 4 + 3 * 2 * 4 * 64 * 4;
    if (P.basis.fb == 1 && (with_sums <= nna::CQL_LDS_TWO / 4 || (words > nna::CQL_LDS_TWO / 4 && with_sums <= nna::CQL_LDS_ONE / 4))) {
      P.shared = (words + 3) / 4 * 4;
      P.lds_floats = std::max(P.lds_floats, with_sums);
    }
    const hipError_t e = nna::launch_cqt_project(P, reinterpret_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
  }
  const hipError_t e = nna::launch_cqt_lowrank(P, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return fail_hip(e, "kernel launch");
  return NNA_OK;
}

// The kernels tap by tap (nna_kernels_short.hip).
// Rows of whole hops: tiles of 64 frames where 80 KB, half a CU's LDS, hold their samples and there are two of them per CU; else tiles of
// 128 frames by columns where there are as many of these, or, where long kernels take the rows, of 64; else 32 or 16 frames, which fill the
// chip sooner.  12 bins, hop 512: 16 frames 7.9, 18.6, 30.2, 53.5 us for 5,500, 17,250, 34,500, 69,000 frames, columns 20.5, 25.2, 29.9, 38.6;
// 24 bins, hop 128: 64 frames 12.1, 15.2, 23.0, 36.4, columns 19.9, 20.3, 25.2, 36.0, 32 frames 9.4, 13.0, 19.6, 31.8; hop 64, 138,000 frames: 47
// with 64, 54 with 32, 60 by columns; 117,200 frames, kernels of 4,336 taps, hop 256 and 128: 64 by columns 401, 358, 128 with half of their
// frames 478, 472.
// Rows of own taps share nothing that a longer run of frames would keep: by columns from 300 tiles of 128 on (12 bins, 128 samples a frame,
// 20,000, 60,000, 120,000 frames: columns 10.1, 12.7, 18.6, 64 frames 8.8, 16.1, 30.3, 32 frames 8.1, 14.3, 24.1; 256 samples: columns 16.5, 21.9,
// 31.1, 64 by columns 14.0, 27.6, 47.7; 960: 45,000 frames 57.3, 53.2).
// 16 frames that take more than 80 KB leave a CU one workgroup: up to 1,024 tiles, or where columns cannot be (25,000 frames of 1,024 samples: 67 us,
// 64 by columns 53; 11,800 of two items of 800: 33, 53).  Against cqt_kernel they take, hops 1,000 to 1,500, 60,000 frames and more: kernels of 1.05
// hops 0.9 .. 1.6 of its time, 1.6 hops 0.95 .. 1.1, 2.5 hops 0.8; two items 1.6 hops 1.1 .. 1.3, 2 hops 1.06, 2.5 hops 1.02, 3.5 hops 0.83.
// Hops that are no multiple of 32, 60,000 frames of 36 bins of up to 4,360 taps: hop 80, 32 frames 228 us, hop 240, 16 frames 423, cqt_kernel 757, 799.
// A tile that holds less than three quarters of its frames is left to the next one.  False: not a launch for this kernel.
bool shape_short(const nna_plan* sub, long long n_frames, long long T, nna::ShortParams& P) {
  auto fit = [&](int form, size_t lds) { return fit_short(sub, n_frames, T, form, lds, P); };
  auto many = [&](long long tiles) { return P.n_ft * P.n_items >= tiles; };
  const bool apart = sub->h_sitems[0].jspan == 1;
  int most = 0;
  long long longest = 0;
  for (const nna::ShortItem& it : sub->h_sitems) most = std::max(most, it.width);
  for (int k = 0; k < sub->n_bins; ++k) longest = std::max(longest, sub->row_e[2 * k] - sub->row_s[2 * k]);
  if (!apart && fit(nna::SHORT_64, 80 * 1024) && many(512)) return true;
  if (fit(nna::SHORT_COLUMNS, 0) && many(apart && most <= 512 ? 300 : 512)) return true;
  if (fit(nna::SHORT_COLUMNS_64, 80 * 1024) && many(512)) return true;
  if (fit(nna::SHORT_32, 80 * 1024) && many(256)) return true;
  if (fit(nna::SHORT_16, 80 * 1024)) return true;
  const bool one = fit(nna::SHORT_16, nna::SHORT_LDS);
  if (one && !many(1024)) return true;
  if (fit(nna::SHORT_COLUMNS_64, 80 * 1024)) return true;
  return one && fit(nna::SHORT_16, nna::SHORT_LDS) && (!many(6144) || 10 * longest > (P.n_items == 1 ? 15LL : 21LL) * sub->hop);
}

nna_status run_conv_short(const nna_plan* sub, const float* x, long long B, long long L, long long T, float* out,
                          long long out_wave_stride, int row_offset, nna::ShortParams& P, void* hip_stream) {
  P.g = make_geom(sub, x, B, L, T);
  set_short(sub, P);
  P.out = out + (long long)row_offset * T;
  P.out_wave_stride = out_wave_stride;
  P.fmt = sub->fmt;
  const hipError_t e = nna::launch_cqt_short(P, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return fail_hip(e, "kernel launch");
  return NNA_OK;
}

hipError_t launch_conv(const nna_plan* sub, const nna::CqtParams& P, hipStream_t stream) {
  if (sub->d_wrm) {
    const long long T = P.g.T, rows = nna::CQW_FRAMES + (1 + (nna::CQW_FRAMES - 1 + T - 1) / T) * (sub->few_jspan - 1);
    const bool tiled = sub->d_few_groups && rows <= nna::CQW_ROWS;
    if (P.g.n_frames < (tiled || !sub->sliding || P.tile_frames < 128 ? sub->few_frames : sub->few_frames_untiled))
      return nna::launch_cqt_few(P, sub->d_row_lo, sub->d_row_hi, sub->d_few_groups, sub->d_few_first, tiled ? (int)rows : 0, stream);
  }
  return nna::launch_cqt(P, stream);
}

// one launch of the CQT kernel: `sub`'s bank over T frames of each of the B waveforms in x
nna_status run_conv(const nna_plan* sub, const float* x, long long B, long long L, long long T, float* out,
                    long long out_wave_stride, int row_offset, void* hip_stream, bool may_fold, float* keep, void* workspace,
                    size_t workspace_bytes) {
  if (sub->runs_lowrank()) {
    nna::CqlParams Q;
    std::memset(&Q, 0, sizeof(Q));
    if (shape_lowrank(sub, B * T, T, Q)) return run_conv_lowrank(sub, x, B, L, T, out, out_wave_stride, row_offset, Q, hip_stream, workspace, workspace_bytes);
  }
  if (sub->runs_short()) {
    nna::ShortParams Q;
    std::memset(&Q, 0, sizeof(Q));
    if (shape_short(sub, B * T, T, Q)) return run_conv_short(sub, x, B, L, T, out, out_wave_stride, row_offset, Q, hip_stream);
  }
  const int extra = (sub->max_jspan - 1) * sub->row_step;
  const int M = pick_tile_frames(CQ_FRAMES, T, extra, CQ_LDS_ROWS_MAX);
  if (may_fold && sub->runs_cqfold()) {
    // the folded kernel does half the work per frame; its tiles hold fewer rows, so batches of very short
    // waveforms (many waveform segments, each with its overlap rows, in one tile) can leave it the smaller tile
    const int Mf = pick_tile_frames(CQ_FRAMES, T, sub->q_max_jspan - 1, nna::CQF_LDS_ROWS);
    if (Mf >= 1 && 2 * Mf >= M) return run_conv_fold(sub, x, B, L, T, out, out_wave_stride, row_offset, Mf, hip_stream);
  }
  if (M < 1) return fail(NNA_ERR_UNSUPPORTED, "frame tile does not fit in LDS");
  nna::CqtParams P;
  std::memset(&P, 0, sizeof(P));
  P.g = make_geom(sub, x, B, L, T);
  P.tap_stride = sub->tap_stride;
  P.row_step = sub->row_step;
  P.bank = reinterpret_cast<const float4*>(sub->d_bank);
  P.items = sub->d_items;
  P.chunks = sub->d_chunks;
  P.out = out;
  P.out_wave_stride = out_wave_stride;
  P.row_offset = row_offset;
  P.n_items = (int)sub->h_items.size();
  P.n_chunks = sub->n_chunks;
  P.n_bins = sub->n_bins;
  P.fmt = sub->fmt;
  P.keep = keep;
  P.rows_pad = sub->rows_pad;
  P.tile_frames = M;
  const long long nseg = 1 + (M - 1 + T - 1) / T;
  P.lds_rows = (int)((M + nseg * extra + 63) / 64 * 64);  // whole loader passes of 64 rows (<= CQ_LDS_ROWS_MAX)
  P.n_ft = (P.g.n_frames + M - 1) / M;
  hipError_t e = launch_conv(sub, P, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return fail_hip(e, "kernel launch");
  return NNA_OK;
}

// A plan with frequency-domain kernels: both stages as one bank while the kernels are fixed -- 4 n_bins K flops per frame where
// the two stages take 2 K^2 for every 64 or 96 bins (16 x 220,500 samples, 84 bins, K = 16,384: 120 ms -> 566 us) -- and the
// two-stage kernel once they are trainable, each stage then being a weight of its own.
nna_status run_cqt1992(const nna_plan* plan, const float* x, long long B, long long L, long long T, float* out,
                       long long out_wave_stride, int row_offset, void* hip_stream) {
  if (!plan->runs_composed())
    return run_stft_core(plan, NNA_KIND_CQT1992, x, B, L, T, out, out_wave_stride, row_offset, hip_stream);
  DeviceGuard guard;
  hipError_t e = guard.enter(plan->device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  return run_conv(plan->composed, x, B, L, T, out, out_wave_stride, row_offset, hip_stream);
}

// one decimation step: y[B, Ln] from x[B, L], Ln = ceil(L / 2) (arguments checked by the caller)
nna_status run_fir(const nna_plan* fir, const float* x, long long B, long long L, float* y, long long Ln, void* hip_stream) {
  nna::FirParams P;
  std::memset(&P, 0, sizeof(P));
  P.L = L;
  P.Ln = Ln;
  P.he = fir->d_fir_he;
  P.ho = fir->d_fir_ho;
  P.hp = fir->d_fir_planes;
  P.ne = (int)fir->h_fir_he.size();
  P.no = (int)fir->h_fir_ho.size();
  P.ve0 = fir->fir_ve0;
  P.vo0 = fir->fir_vo0;
  const int vmin = std::min(P.ve0, P.vo0), vend = std::max(P.ve0 + P.ne, P.vo0 + P.no);
  P.lds_stream = (nna::FIR_TILE + (vend - vmin) + 16) * 9 / 8 + 8;  // one float of padding per eight samples
  // the grid's second dimension holds at most 65,535 waveforms
  for (long long b0 = 0; b0 < B; b0 += 65535) {
    P.B = std::min(B - b0, 65535LL);
    P.x = x + b0 * L;
    P.y = y + b0 * Ln;
    P.vec2 = ((reinterpret_cast<uintptr_t>(P.x) & 7) == 0 && (L % 2 == 0 || P.B == 1)) ? 1 : 0;
    P.vec4_out = ((reinterpret_cast<uintptr_t>(P.y) & 15) == 0 && (Ln % 4 == 0 || P.B == 1)) ? 1 : 0;
    const hipError_t e = nna::launch_fir_decimate(P, reinterpret_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
  }
  return NNA_OK;
}

inline size_t ws_round(long long floats) { return ((size_t)floats * sizeof(float) + 255) / 256 * 256; }

// lengths of the waveform at every octave; false if some octave is too short for its padding
bool cqt2010_lengths(const nna_plan* plan, long long L, long long (&La)[MAX_OCTAVES]) {
  const int n_oct = (int)plan->octave.size();
  long long l = L;
  for (int a = 0; a < n_oct; ++a) {
    La[a] = l;
    if (l < 4 || l <= plan->pad) return false;             // mirror reflection of the CQT kernels
    if (a + 1 < n_oct && l < plan->fir->K) return false;   // and of the filter's frames
    l = (l + 1) / 2;
  }
  return true;
}

}  // namespace host
}  // namespace nna

using namespace nna::host;

// =======================================================================================
// C ABI: transforms
// =======================================================================================
extern "C" {

nna_status nna_cqt1992(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev, void* hip_stream) {
  long long T = 0;
  nna_status s = check_call(plan, NNA_KIND_CQT1992, x_dev, B, L, out_dev, &T);
  if (s != NNA_OK) return s;
  return run_cqt1992(plan, x_dev, B, L, T, out_dev, (long long)plan->out_rows() * T, 0, hip_stream);
}

nna_status nna_cqt2010v2_workspace(const nna_plan* plan, long long B, long long L, size_t* bytes) {
  if (!plan || !bytes) return fail(NNA_ERR_INVALID_ARG, "plan / bytes is NULL");
  if (plan->kind != NNA_KIND_CQT2010V2 && plan->kind != NNA_KIND_CQT2010)
    return fail(NNA_ERR_INVALID_ARG, "plan was built for a different transform");
  if (B < 1 || L < 1) return fail(NNA_ERR_SHAPE, "B and L must be >= 1");
  const int n_oct = (int)plan->octave.size();
  const long long L1 = (L + 1) / 2, L2 = (L1 + 1) / 2;
  *bytes = (n_oct > 1 ? ws_round(B * L1) : 0) + (n_oct > 2 ? ws_round(B * L2) : 0);
  return NNA_OK;
}

// the octave loop of both downsampling plans (time-domain or frequency-domain kernels per octave)
static nna_status run_octaves(const nna_plan* plan, int kind, const float* x_dev, long long B, long long L,
                              float* out_dev, void* workspace_dev, size_t workspace_bytes, void* hip_stream) {
  if (!plan) return fail(NNA_ERR_INVALID_ARG, "plan is NULL");
  if (plan->kind != kind) return fail(NNA_ERR_INVALID_ARG, "plan was built for a different transform");
  if (!x_dev || !out_dev) return fail(NNA_ERR_INVALID_ARG, "x_dev / out_dev is NULL");
  if (plan->device < 0) return fail(NNA_ERR_UNSUPPORTED, "host-only plan (device = -1) cannot run transforms");
  if (B < 1) return fail(NNA_ERR_SHAPE, "B must be >= 1");
  long long La[MAX_OCTAVES];
  if (L < 1 || !cqt2010_lengths(plan, L, La))
    return fail(NNA_ERR_SHAPE, "L is too short: every octave's waveform must exceed the reflection padding, and all but the lowest hold one frame of the decimation filter");
  const long long T = 1 + L / plan->hop;
  if (T > 0x7fffffffLL / 4 || L > 0x7fffffffLL - 4LL * plan->K - 64 || B > 0x7fffffffLL || B > (1LL << 40) / T)
    return fail(NNA_ERR_SHAPE, "batch too large");
  size_t need = 0;
  nna_status s = nna_cqt2010v2_workspace(plan, B, L, &need);
  if (s != NNA_OK) return s;
  if (need > 0 && (!workspace_dev || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace_dev) & 15)))
    return fail(NNA_ERR_INVALID_ARG, "workspace_dev is NULL, misaligned or smaller than nna_cqt2010v2_workspace asks for");
  const int n_oct = (int)plan->octave.size();
  // every launch of the call must fit before the first one is enqueued
  for (int a = 0; a < n_oct; ++a) {
    const nna_plan* sub = plan->octave[a]->runs_composed() ? plan->octave[a]->composed : plan->octave[a];
    const int lds_rows = sub->kind == NNA_KIND_CQT1992 && sub->lin_blocks == 6 ? nna::ST_LDS_ROWS_WIDE : ST_LDS_ROWS;
    const int M = sub->kind == NNA_KIND_CQT ? pick_tile_frames(CQ_FRAMES, T, (sub->max_jspan - 1) * sub->row_step, CQ_LDS_ROWS_MAX)
                                             : pick_tile_frames(ST_FRAMES, T, sub->nj - 1, lds_rows);
    if (M < 1) return fail(NNA_ERR_UNSUPPORTED, "frame tile does not fit in LDS");
  }
  float* buf[2] = {static_cast<float*>(workspace_dev), nullptr};
  if (n_oct > 2) buf[1] = reinterpret_cast<float*>(static_cast<char*>(workspace_dev) + ws_round(B * ((L + 1) / 2)));
  DeviceGuard guard;
  hipError_t e = guard.enter(plan->device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  // The filter chain x_0 -> x_1 -> ... runs on the caller's stream; octave a's kernels need x_a only and go to one of the
  // plan's two streams (even / odd octaves), so they run beside the next filter steps and beside each other: the
  // filter alone keeps the matrix pipe a third busy and waits for more than half of its time, and the deep octaves' launches are too
  // small to fill the chip alone.  Every stream is back on the caller's before the call returns, so the call still
  // is one piece of work on that stream (under stream capture: a fork and a join).
  hipStream_t main_stream = static_cast<hipStream_t>(hip_stream);
  const bool forked = n_oct > 1 && plan->oct_stream[0] != nullptr;
  std::unique_lock<std::mutex> lock(plan->oct_mutex, std::defer_lock);
  if (forked) {
    lock.lock();
    if ((e = hipEventRecord(plan->ev_fork, main_stream)) != hipSuccess) return fail_hip(e, "hipEventRecord");
    for (hipStream_t st : plan->oct_stream)
      if ((e = hipStreamWaitEvent(st, plan->ev_fork, 0)) != hipSuccess) return fail_hip(e, "hipStreamWaitEvent");
  }
  int launched = 0;  // octaves whose kernels were enqueued on the plan's streams
  // the caller's stream waits for the last octave enqueued on each of the plan's streams (also on an error path)
  auto join = [&]() -> hipError_t {
    hipError_t r = hipSuccess;
    for (int a = std::max(0, launched - 2); a < launched; ++a) {
      const hipError_t w = hipStreamWaitEvent(main_stream, plan->ev_oct[a], 0);
      if (r == hipSuccess) r = w;
    }
    return r;
  };
  const float* cur = x_dev;
  for (int a = 0; a < n_oct; ++a) {
    int lo, hi;
    octave_bins(plan->n_bins, plan->bpo, a, lo, hi);
    // the octave's rows inside each waveform's output (the complex format writes two rows per bin)
    const int row0 = plan->fmt == NNA_OUT_COMPLEX ? 2 * lo : lo;
    hipStream_t st = forked ? plan->oct_stream[a & 1] : main_stream;
    if (forked && a >= 1 && (e = hipStreamWaitEvent(st, plan->ev_fir[a], 0)) != hipSuccess) {  // x_a is complete
      (void)join();
      return fail_hip(e, "hipStreamWaitEvent");
    }
    if (kind == NNA_KIND_CQT2010V2)
      s = run_conv(plan->octave[a], cur, B, La[a], T, out_dev, (long long)plan->out_rows() * T, row0, st);
    else
      s = run_cqt1992(plan->octave[a], cur, B, La[a], T, out_dev, (long long)plan->out_rows() * T, row0, st);
    if (forked) {
      e = hipEventRecord(plan->ev_oct[a], st);
      if (e == hipSuccess) launched = a + 1;
      if (s == NNA_OK && e != hipSuccess) s = fail_hip(e, "hipEventRecord");
    }
    if (s != NNA_OK) {
      if (forked) (void)join();
      return s;
    }
    if (a + 1 < n_oct) {
      float* dst = buf[a & 1];
      const long long Ln = La[a + 1];
      // dst held x_(a-1): octave a-1 must have read it
      if (forked && a >= 2 && (e = hipStreamWaitEvent(main_stream, plan->ev_oct[a - 1], 0)) != hipSuccess) {
        (void)join();
        return fail_hip(e, "hipStreamWaitEvent");
      }
      s = run_fir(plan->fir, cur, B, La[a], dst, Ln, main_stream);
      if (s == NNA_OK && forked && (e = hipEventRecord(plan->ev_fir[a + 1], main_stream)) != hipSuccess)
        s = fail_hip(e, "hipEventRecord");
      if (s != NNA_OK) {
        if (forked) (void)join();
        return s;
      }
      cur = dst;
    }
  }
  if (forked && (e = join()) != hipSuccess) return fail_hip(e, "hipStreamWaitEvent");
  return NNA_OK;
}

nna_status nna_cqt2010v2(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev,
                         void* workspace_dev, size_t workspace_bytes, void* hip_stream) {
  return run_octaves(plan, NNA_KIND_CQT2010V2, x_dev, B, L, out_dev, workspace_dev, workspace_bytes, hip_stream);
}

nna_status nna_cqt2010v2_static(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev,
                                void* hip_stream) {
  if (!plan) return fail(NNA_ERR_INVALID_ARG, "plan is NULL");
  if (plan->kind != NNA_KIND_CQT2010V2) return fail(NNA_ERR_INVALID_ARG, "plan was built for a different transform");
  if (plan->device < 0) return fail(NNA_ERR_UNSUPPORTED, "host-only plan (device = -1) cannot run transforms");
  if (B < 1 || L < 1) return fail(NNA_ERR_SHAPE, "B and L must be >= 1");
  // the workspace the batch needs, before any size is turned into bytes that could wrap around
  if (B > (long long)NNA_STATIC_SCRATCH_BYTES || L > (long long)NNA_STATIC_SCRATCH_BYTES)
    return fail(NNA_ERR_SHAPE, "batch too large for the library's static workspace (NNA_STATIC_SCRATCH_BYTES)");
  size_t need = 0;
  nna_status s = nna_cqt2010v2_workspace(plan, B, L, &need);
  if (s != NNA_OK) return s;
  if (need > (size_t)NNA_STATIC_SCRATCH_BYTES) {
    char msg[200];
    std::snprintf(msg, sizeof msg,
                  "this batch needs %zu bytes of workspace; the library's static workspace holds %zu "
                  "(NNA_STATIC_SCRATCH_BYTES): use nna_cqt2010v2 with a caller-owned workspace",
                  need, (size_t)NNA_STATIC_SCRATCH_BYTES);
    return fail(NNA_ERR_SHAPE, msg);
  }
  void* ws = scratch_of(plan->device);  // found when the plan was built, with its device current
  if (!ws) return fail(NNA_ERR_HIP, "the static workspace of the plan's device was never located");
  return run_octaves(plan, NNA_KIND_CQT2010V2, x_dev, B, L, out_dev, ws, (size_t)NNA_STATIC_SCRATCH_BYTES, hip_stream);
}

nna_status nna_cqt2010(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev,
                       void* workspace_dev, size_t workspace_bytes, void* hip_stream) {
  return run_octaves(plan, NNA_KIND_CQT2010, x_dev, B, L, out_dev, workspace_dev, workspace_bytes, hip_stream);
}

nna_status nna_out_shape(const nna_plan* plan, long long B, long long L, long long* n_bins, long long* n_frames) {
  if (!plan) return fail(NNA_ERR_INVALID_ARG, "plan is NULL");
  if (B < 1) return fail(NNA_ERR_SHAPE, "B must be >= 1");
  if (plan->kind == NNA_KIND_CQT2010V2 || plan->kind == NNA_KIND_CQT2010) {
    long long La[MAX_OCTAVES];
    if (L < 1 || !cqt2010_lengths(plan, L, La))
      return fail(NNA_ERR_SHAPE, "L is too short: every octave's waveform must exceed the reflection padding, and all but the lowest hold one frame of the decimation filter");
    if (n_bins) *n_bins = plan->out_rows();
    if (n_frames) *n_frames = 1 + L / plan->hop;
    return NNA_OK;
  }
  if (L < 4) return fail(NNA_ERR_SHAPE, "L must be at least 4 samples");
  const long long T = frames_of(plan, L);
  if (T < 1) return fail(NNA_ERR_SHAPE, plan->center ? "L must exceed the reflection padding (K/2)" : "L is shorter than one window");
  if (n_bins) *n_bins = plan->out_rows();
  if (n_frames) *n_frames = T;
  return NNA_OK;
}

nna_status nna_stft(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev, void* hip_stream) {
  return run_stft_like(plan, NNA_KIND_STFT, x_dev, B, L, out_dev, hip_stream);
}

nna_status nna_mel(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev, void* hip_stream) {
  return run_stft_like(plan, NNA_KIND_MEL, x_dev, B, L, out_dev, hip_stream);
}

nna_status nna_mel_with_stft(const nna_plan* plan, const float* x_dev, long long B, long long L, float* mel_dev,
                             float* spec_dev, void* hip_stream) {
  if (!spec_dev) return fail(NNA_ERR_INVALID_ARG, "spec_dev is NULL");
  long long T = 0;
  nna_status s = check_call(plan, NNA_KIND_MEL, x_dev, B, L, mel_dev, &T);
  if (s != NNA_OK) return s;
  if (plan->precision != NNA_PREC_F32) return fail(NNA_ERR_UNSUPPORTED, "float32 plans only");
  return run_stft_core(plan, NNA_KIND_MEL, x_dev, B, L, T, mel_dev, 0, 0, hip_stream, spec_dev);
}

nna_status nna_cqt(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev, void* hip_stream) {
  long long T = 0;
  nna_status s = check_call(plan, NNA_KIND_CQT, x_dev, B, L, out_dev, &T);
  if (s != NNA_OK) return s;
  DeviceGuard guard;
  hipError_t e = guard.enter(plan->device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  return run_conv(plan, x_dev, B, L, T, out_dev, (long long)plan->out_rows() * T, 0, hip_stream, true);
}

// the plan whose kernels a call of nna_cqt or nna_cqt1992 applies at one rate, or NULL
static const nna_plan* one_rate_plan(const nna_plan* plan) {
  if (plan->kind == NNA_KIND_CQT) return plan;
  return plan->kind == NNA_KIND_CQT1992 && plan->runs_composed() ? plan->composed : nullptr;
}

nna_status nna_cqt_workspace(const nna_plan* plan, long long B, long long L, size_t* bytes) {
  if (!plan || !bytes) return fail(NNA_ERR_INVALID_ARG, "plan / bytes is NULL");
  if (plan->kind != NNA_KIND_CQT && plan->kind != NNA_KIND_CQT1992) return fail(NNA_ERR_INVALID_ARG, "plan was built for a different transform");
  const long long T = B < 1 ? 0 : frames_of(plan, L);
  if (T < 1) return fail(NNA_ERR_SHAPE, "no frames");
  const nna_plan* sub = one_rate_plan(plan);
  *bytes = sub && plan->device >= 0 ? lowrank_workspace(sub, B, L, T) : 0;
  return NNA_OK;
}

nna_status nna_cqt_in_workspace(const nna_plan* plan, const float* x_dev, long long B, long long L, float* out_dev, void* workspace_dev,
                                size_t workspace_bytes, void* hip_stream) {
  if (!plan) return fail(NNA_ERR_INVALID_ARG, "plan is NULL");
  const nna_plan* sub = one_rate_plan(plan);
  if (!sub || !workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 15))
    return plan->kind == NNA_KIND_CQT1992 ? nna_cqt1992(plan, x_dev, B, L, out_dev, hip_stream) : nna_cqt(plan, x_dev, B, L, out_dev, hip_stream);
  long long T = 0;
  nna_status s = check_call(plan, plan->kind, x_dev, B, L, out_dev, &T);
  if (s != NNA_OK) return s;
  DeviceGuard guard;
  hipError_t e = guard.enter(plan->device);
  if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
  return run_conv(sub, x_dev, B, L, T, out_dev, (long long)plan->out_rows() * T, 0, hip_stream, plan->kind == NNA_KIND_CQT, nullptr, workspace_dev,
                  workspace_bytes);
}
}  // extern "C"
