// Backward kernels of the RFF linear attention (Eq.(linear att) with the
// Flexformer feature maps of Eq.(phi_n) / Eq.(phi_non)).  The paper gives no
// backward; this is the derivative of the forward:
//
//   [num|den]_i = sum_j a_ij [V_j ; 1],  a_ij = phi(Q_i).phi(K_j)  (j <= i if causal)
//   G_i = [dO_i ; -delta_i] / den_i,     delta_i = dO_i . O_i
//   dphi(Q_i) = S'_i G_i,   S'_i = sum_{j(<=i)} phi(K_j) [V_j;1]^T
//   dphi(K_j) = R'_j [V_j;1], R'_j = sum_{i(>=j)} phi(Q_i) G_i^T
//   dV_j = (R'_j^T phi(K_j))[:dv]
// then the feature-map chain rule (frequencies and norm factor exp(||x||^2/c)).
//
// Kernels (per (b,h) slice, sequence split into segments like the forward):
//   k_bwd_prepass : segment-local S'^T (key side) and R'^T (query side), and the
//                   per-token scalars 1/den_i, delta_i,
//   k_state_scan  : prefix of S' and suffix of R' over segments,
//   k_bwd_dq      : ascending chunk sweep carrying S'; dQ and the query-side
//                   frequency-gradient partials (flex_bwd_dq.hip),
//   k_bwd_dkv     : descending chunk sweep carrying R'; dK, dV, the key-side
//                   frequency-gradient partials and dtau partials,
//   k_bwd_reduce  : fixed-order sums of the partials into dW1, dW2, dtau.
// Waves split the frequencies in the work on features and states, and the output
// tiles in the products over all features.  Both states are held as accumulator
// tiles with value columns as rows ([dv' x features]).
#include "flex_bwd_common.hpp"

namespace flex {

// ---------------------------------------------------------------------------
// Pre-pass: segment-local S'^T = sum [V;1]^T-rows x phi(K) and
// R'^T = sum [dO;-delta]^T-rows x phi(Q)/den; per-token 1/den and delta.
// ---------------------------------------------------------------------------
// Launched where the forward's segment states are not passed in (with them the dQ
// sweep does the query-side work).
// The pre-pass forms sums over a segment and per-token scalars only, so at
// d <= 64 it walks the segment in 64-token chunks (a backward segment is a
// whole number of them: it spans the forward's 64-token chunks), not the
// sweeps' 32; at d = 128 the double-buffered staging of 64 rows would not fit
// in LDS.
template <class T, int D, int FW, int NW, bool NS, bool MASK = false>
__global__ __launch_bounds__(NW * WAVE) void k_bwd_prepass(BwdArgs a) {
  constexpr int PCH = D <= 64 ? CHUNK : BWD_CHUNK;
  typedef Shape<T, D, FW, NW, NS, PCH> SH;
  static_assert(PCH % BWD_CHUNK == 0 && CHUNK % PCH == 0, "pre-pass chunks hold whole sweep chunks");
  typedef typename Io<T>::type IO;
  typedef RowStage<IO, D, SH::NT, SH::CH> StX;
  typedef RowStage<IO, SH::DV, SH::NT, SH::CH> StV;
  // staging (and the per-token scalars) double-buffered by chunk parity
  __shared__ __attribute__((aligned(16))) IO XQ2[2][StX::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XK2[2][StX::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XDO2[2][StV::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XO2[2][StV::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XV2[2][StV::LDS_ELEMS];
  __shared__ float GS2[2][SH::CH][2];
  __shared__ float DEN2[2][SH::CH];
  __shared__ typename StX::Ssq SSQ2[2][SH::CH], SSK2[2][SH::CH];
  // per-token feature scales: s e(k) for keys, s e(q) / den for queries
  __shared__ __attribute__((aligned(16))) float SCK2[2][SH::CH], SCQ2[2][SH::CH];

  const WgCoord wc = wg_coord(a.segments, a.H, a.BH);
  const int seg = wc.seg, bh = wc.bh, h = bh % a.H;
  const int w = threadIdx.x / WAVE, l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  const int fv = slice_valid<MASK, FW>(a.fvalid, w);
  const int cps = a.chunks_per_seg / (PCH / BWD_CHUNK);   // pre-pass chunks per segment
  const int c0 = seg * cps;
  const int c1 = min(c0 + cps, (a.N + SH::CH - 1) / SH::CH);
  const IO* Q = static_cast<const IO*>(a.Q) + (size_t)bh * a.N * D;
  const IO* K = static_cast<const IO*>(a.K) + (size_t)bh * a.N * D;
  const IO* V = static_cast<const IO*>(a.V) + (size_t)bh * a.N * SH::DV;
  const IO* dO = static_cast<const IO*>(a.dO) + (size_t)bh * a.N * SH::DV;
  const IO* Ob = static_cast<const IO*>(a.O) + (size_t)bh * a.N * SH::DV;
  const float* den = a.den + (size_t)bh * a.N;
  float* gst = a.gstats + (size_t)bh * a.N * 2;

  StX sq, sk;
  StV sv, sdo, so;
  // FUSED: every thread stages the same PER vectors of Q, dO and O (same
  // vectors per row, all threads busy), so the row sums dO . O and ||q||^2
  // come out of the staging registers with lane sums, and the per-token
  // scalars need no barrier of their own.  Each thread then loads den of its
  // own rows; otherwise thread t < CH loads that of row t.
  constexpr bool FUSED = StX::VPR == StV::VPR && StX::NV == StV::NV && StV::NV % SH::NT == 0;
  constexpr int FPER = FUSED ? StV::PER : 1;
  float dn_next[FPER];
#pragma unroll
  for (int i = 0; i < FPER; ++i) dn_next[i] = 0.f;
  auto den_rows = [&](int t0) {
#pragma unroll
    for (int i = 0; i < FPER; ++i) {
      const int t = FUSED ? (int)(threadIdx.x + i * SH::NT) / StV::VPR : (int)(threadIdx.x % SH::CH);
      dn_next[i] = den[min(t0 + t, a.N - 1)];   // rows past N unused
    }
  };
  if (c0 < c1) {
    sq.fetch(Q, c0 * SH::CH, a.N); sk.fetch(K, c0 * SH::CH, a.N);
    sv.fetch(V, c0 * SH::CH, a.N); sdo.fetch(dO, c0 * SH::CH, a.N); so.fetch(Ob, c0 * SH::CH, a.N);
    den_rows(c0 * SH::CH);
  }
  const Frag<T>* wproj = FragBlock<T, D, FW, NS>::proj(a.wfrag, h, NW, w);
  const auto inv_c = inv_c_of<T>(a.tau[h]);

  f32x4 ST[SH::DVT1][SH::FC], RT[SH::DVT1][SH::FC];
#pragma unroll
  for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
    for (int fc = 0; fc < SH::FC; ++fc) { ST[dt][fc] = zero4(); RT[dt][fc] = zero4(); }
  const Frag<T> ones = ones_col01<T>();
  constexpr int TPT = SH::NT / SH::CH;  // threads per token for the row reductions

  // projection fragments, reloaded per chunk ahead of the staging barriers
  FreqSlice<T, D, FW, NS> fs;
  for (int c = c0; c < c1; ++c) {
    // This chunk's buffers.  They need no barrier before they are written:
    // the chunk that last read them (two back) is separated from this point
    // by the previous chunk's barriers.
    const int par = (c - c0) & 1;
    IO* XQ = XQ2[par];
    IO* XK = XK2[par];
    IO* XDO = XDO2[par];
    IO* XO = XO2[par];
    IO* XV = XV2[par];
    float (*GS)[2] = GS2[par];
    float* DEN = DEN2[par];
    typename StX::Ssq* SSQ = SSQ2[par];
    typename StX::Ssq* SSK = SSK2[par];
    float* SCK = SCK2[par];
    float* SCQ = SCQ2[par];
    const int tok0 = c * SH::CH;
    fs.load_frags(wproj);
    if constexpr (FUSED) {
      // per-token 1/den and delta = dO . O of this thread's rows (rows past N
      // are zero vectors: delta 0)
      float inv[FPER];
      bool ok[FPER];
#pragma unroll
      for (int i = 0; i < FPER; ++i) {
        const int t = (int)(threadIdx.x + i * SH::NT) / StV::VPR;
        ok[i] = tok0 + t < a.N;
        inv[i] = ok[i] ? 1.0f / dn_next[i] : 0.f;
        float dsum = 0.f;
        const uint4 x = sdo.vec(i), y = so.vec(i);
        const IO* ex = reinterpret_cast<const IO*>(&x);
        const IO* ey = reinterpret_cast<const IO*>(&y);
#pragma unroll
        for (int j = 0; j < StV::VEC; ++j) dsum += io_to_float(ex[j]) * io_to_float(ey[j]);
        dsum = lane_sum<StV::VPR>(dsum);
        if (threadIdx.x % StV::VPR == 0) {
          GS[t][0] = inv[i];
          GS[t][1] = ok[i] ? dsum : 0.f;
          if (ok[i]) { gst[(size_t)(tok0 + t) * 2] = inv[i]; gst[(size_t)(tok0 + t) * 2 + 1] = dsum; }
        }
      }
      sq.store_idx(XQ, SCQ, [&](int i, int, auto ssq) { return row_scale(ssq, inv_c, a.s_const, ok[i]) * inv[i]; });
      sdo.store(XDO);
    } else {
      sq.store(XQ, SSQ); sdo.store(XDO); so.store(XO);
      if (threadIdx.x < SH::CH) DEN[threadIdx.x] = dn_next[0];
    }
    if constexpr (FUSED)
      sk.store(XK, SCK, [&](int t, auto ssq) { return row_scale(ssq, inv_c, a.s_const, tok0 + t < a.N); });
    else
      sk.store(XK, SSK);
    sv.store(XV);
    {
      const int t1 = c + 1 < c1 ? tok0 + SH::CH : tok0;   // the last chunk refetches itself (unused)
      sq.fetch(Q, t1, a.N); sk.fetch(K, t1, a.N);
      sv.fetch(V, t1, a.N); sdo.fetch(dO, t1, a.N); so.fetch(Ob, t1, a.N);
      den_rows(t1);
    }
    __syncthreads();
    // per-token 1/den and delta = dO . O (FUSED: done above)
    if constexpr (!FUSED) {
      const int t = threadIdx.x / TPT, part = threadIdx.x % TPT;
      float s = 0.f;
      for (int cidx = part; cidx < SH::DV; cidx += TPT)
        s += io_to_float(XDO[t * StV::LD + cidx]) * io_to_float(XO[t * StV::LD + cidx]);
      s = lane_sum<TPT>(s);
      if (part == 0) {
        const bool ok = tok0 + t < a.N;
        const float inv = ok ? 1.0f / DEN[t] : 0.f;
        GS[t][0] = inv;
        GS[t][1] = ok ? s : 0.f;
        SCK[t] = row_scale(SSK[t], inv_c, a.s_const, ok);
        SCQ[t] = row_scale(SSQ[t], inv_c, a.s_const, ok) * inv;
        if (ok) { gst[(size_t)(tok0 + t) * 2] = inv; gst[(size_t)(tok0 + t) * 2 + 1] = s; }
      }
      __syncthreads();
    }
    // both feature maps enter only the token sums: token-row features, no
    // transpose; the key side and the query side one after the other
#pragma unroll
    for (int ks = 0; ks < SH::KT; ++ks) {
      // value-side operands: rows = value columns, k = chunk tokens
      {
        Frag<T> vt[SH::DVT1], pk[SH::FC];
#pragma unroll
        for (int dt = 0; dt < SH::DVT; ++dt) vt[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XV), StV::LD, 32 * ks + 4 * g, 32 * ks + 16 + 4 * g, dt * 16);
        vt[SH::DVT] = ones;
        feature_frags_rows<T, D, FW, NS, StX::LD>(fs, XK, SCK, ks, pk, fv);
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
          for (int dt = 0; dt < SH::DVT1; ++dt) mma(ST[dt][fc], vt[dt], pk[fc]);
      }
      {
        Frag<T> gt[SH::DVT1], pq[SH::FC];
#pragma unroll
        for (int dt = 0; dt < SH::DVT; ++dt) gt[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XDO), StV::LD, 32 * ks + 4 * g, 32 * ks + 16 + 4 * g, dt * 16);
        gt[SH::DVT] = delta_rows<T>(GS, ks);
        feature_frags_rows<T, D, FW, NS, StX::LD>(fs, XQ, SCQ, ks, pq, fv);
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
          for (int dt = 0; dt < SH::DVT1; ++dt) mma(RT[dt][fc], gt[dt], pq[fc]);
      }
    }
  }
  float* so_ = a.sstate + ((size_t)bh * a.segments + seg) * SH::STATE;
  float* ro_ = a.rstate + ((size_t)bh * a.segments + seg) * SH::STATE;
#pragma unroll
  for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
    for (int fc = 0; fc < SH::FC; ++fc) {
      *reinterpret_cast<f32x4*>(so_ + state_off<SH>(w, dt, fc, l)) = ST[dt][fc];
      *reinterpret_cast<f32x4*>(ro_ + state_off<SH>(w, dt, fc, l)) = RT[dt][fc];
    }
}

// ---------------------------------------------------------------------------
// dK, dV: descending sweep with the query-side suffix state R'.
//
// A chunk has three intervals between two barriers, the last one running on
// into the next chunk's first:
//   1  (waves split the frequencies) phi(Q)/den, phi(K) and the bf16 copy of R'
//      to LDS; the R' share of dphi(K); three waves form the tiles of the
//      intra-chunk matrix M = dO V^T - delta
//   2  (frequencies) the M share of dphi(K), the R' update, the chain rule, dP
//      to LDS, the next chunk's rows to LDS; (output tiles) the R' share of dV
//      over all features; three waves form the tiles of the intra-chunk matrix
//      A = phi(Q)/den phi(K)^T
//   3  (output tiles) the A share of dV, dK = dP W'; (frequencies) dW' += dP^T K
// So M and A are formed once per workgroup and no partial sum of dV crosses
// waves; dW' stays in registers for the whole sweep.
//
// Bound by latency and LDS traffic: matrix and vector issue each take a third
// of the time, and leaving any one product out gains 3 to 8 %.  So what counts
// is two waves per SIMD (8 waves of 16 frequencies at d = 64, m = 128; two
// workgroups of 4 at m = 64) within 256 registers, and few LDS accesses.  us per
// pass before (dV partials of every wave summed through LDS, dW' there too, 4
// waves of 32 frequencies at m = 128) and after: training step d = 64, m = 128
// (B*H = 32, N = 8192) 469 and 424, d = 128, m = 256 2561 and 2439, encoder
// training (non-causal m = 64, B*H = 64, N = 4000) 253 and 232, then 209 with two
// workgroups per CU.  (A as hi + lo costs 3 of these us at m = 128.)
// ---------------------------------------------------------------------------
// ACC: add dK and dV to the values an earlier frequency group stored.  The
// old values are loaded ahead of the next chunk's prefetch, so waiting for
// them never waits for that prefetch.
template <class T, int D, int FW, int NW, bool NS, bool CAUSAL, bool ACC, bool MASK = false>
__global__ __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(bwd_waves_per_eu(IsBf16<T>::value, D))))
void k_bwd_dkv(BwdArgs a) {
  typedef Shape<T, D, FW, NW, NS, BWD_CHUNK> SH;
  typedef typename Io<T>::type IO;
  // With at least two threads per 16-byte vector of a chunk's rows, half of the
  // waves stage K and Q and the other half V and dO.
  constexpr int HALVES = 2 * SH::CH * D * (int)sizeof(IO) / 16 <= SH::NT ? 2 : 1;
  constexpr int NTH = SH::NT / HALVES;
  typedef RowStage<IO, D, NTH, SH::CH> StX;
  typedef StX StV;
  static_assert(D == SH::DV, "one stage type");
  typedef WTSlice<T, D, FW, NS> WTS;
  constexpr int DT = D / 16;
  constexpr int NFT = SH::M / 16;                // frequency tiles of all waves
  constexpr int KG = (SH::DVT1 + 1) / 2;         // k-steps over [V | 1]
  constexpr int NOT = (DT * SH::TT + NW - 1) / NW;   // dV (and dK) tiles per wave (at most)
  constexpr int RLP = SH::DV + 4;                // row stride of the bf16 R' copy, [feature][value col]
  constexpr int NDX = FragBlock<T, D, FW, NS>::NT_ * WAVE;   // dX fragments per wave
  static_assert(SH::TT == 2 && SH::KT == 1 && NW >= 4, "32-token chunks, three waves for the intra-chunk tiles");
  // rows read in interval 1 only (Q, V) need one staging buffer (stored in
  // interval 2), those read in interval 3 too (K, dO) two, by chunk parity
  __shared__ __attribute__((aligned(16))) IO XQ[CAUSAL ? StX::LDS_ELEMS : 8];
  __shared__ __attribute__((aligned(16))) IO XK2[2][StX::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XV[StV::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XDO2[CAUSAL ? 2 : 1][CAUSAL ? StV::LDS_ELEMS : 8];
  __shared__ FragLds<T> PT[CAUSAL ? SH::TT : 1][CAUSAL ? NFT : 1];   // phi(Q)/den, operand fragments
  __shared__ FragLds<T> DP[SH::TT][NW * WTS::KP];   // dP, operand fragments (k = pairs of projection row tiles)
  __shared__ __attribute__((aligned(16))) T RL[NW][SH::FC * 16 * RLP];   // R' copy
  __shared__ Frag<T> PK[SH::TT][NFT][WAVE];      // phi(K), operand fragments
  // M and A: [key tile], k = query tokens; A as a high and a low operand
  // (rounded once over all features it would carry more error than the features)
  constexpr int NSA = IsBf16<T>::value ? 2 : 1;
  __shared__ Frag<T> MP[SH::TT][WAVE], AP[NSA][SH::TT][WAVE];
  // dX fragments of every wave's projection rows: held in registers with four
  // waves (each then has DT / 4 d tiles), in LDS with eight
  constexpr bool DX_LDS = NW > 4;
  constexpr int NDK = DT > NW ? DT / NW : 1;     // d tiles of one wave
  static_assert(DT <= NW ? NW % DT == 0 : DT % NW == 0, "a wave keeps its d tiles");
  __shared__ Frag<T> DXL[DX_LDS ? NW : 1][DX_LDS ? NDX : 1];
  __shared__ __attribute__((aligned(16))) float SCQ[SH::CH], SCK[SH::CH], INV[SH::CH], DEL[SH::CH];
  // -delta as a (hi, lo) pair of operand rows and a row of zeros (delta_frag)
  constexpr int DLD = SH::CH + 8;
  __shared__ __attribute__((aligned(16))) T DLT2[2][3 * DLD];
  __shared__ typename StX::Ssq SSK2[2][SH::CH];
  __shared__ float TRED[SH::NT];
  __shared__ __attribute__((aligned(16))) float GP[SH::CH][NW + 4];   // every wave's share of g

  const WgCoord wc = wg_coord(a.segments, a.H, a.BH);
  const int seg = wc.seg, bh = wc.bh, h = bh % a.H;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  const int fv = slice_valid<MASK, FW>(a.fvalid, w);
  const int c0 = seg * a.chunks_per_seg;
  const int c1 = min(c0 + a.chunks_per_seg, a.nchunks);
  const IO* Q = static_cast<const IO*>(a.Q) + (size_t)bh * a.N * D;
  const IO* K = static_cast<const IO*>(a.K) + (size_t)bh * a.N * D;
  const IO* V = static_cast<const IO*>(a.V) + (size_t)bh * a.N * SH::DV;
  const IO* dO = static_cast<const IO*>(a.dO) + (size_t)bh * a.N * SH::DV;
  const float* gst = a.gstats + (size_t)bh * a.N * 2;
  float* dK = a.dK + (size_t)bh * a.N * D;
  float* dV = a.dV + (size_t)bh * a.N * SH::DV;

  // the non-causal sweep reads no query-side rows: its R' is the total
  const int half = HALVES == 2 ? w / (NW / 2) : 0;
  constexpr int SV = HALVES == 2 ? 0 : 2, SDO = SV + 1;   // K and Q in st[0], st[1]; V and dO here
  StX st[4 / HALVES];
  float2 gs_next = make_float2(0.f, 0.f);
  auto fetch = [&](int t1) {
    st[0].fetch(HALVES == 2 && half ? V : K, t1, a.N);
    if (CAUSAL) st[1].fetch(HALVES == 2 && half ? dO : Q, t1, a.N);
    if (HALVES == 1) st[SV].fetch(V, t1, a.N);
    if (CAUSAL) {
      if (HALVES == 1) st[SDO].fetch(dO, t1, a.N);
      gs_next = load_gs(gst, t1, a.N, SH::CH, StX::tid());
    }
  };
  if (c0 < c1) fetch((c1 - 1) * SH::CH);
  const Frag<T>* wproj = FragBlock<T, D, FW, NS>::proj(a.wfrag, h, NW, w);
  const auto inv_c = inv_c_of<T>(a.tau[h]);

  f32x4 RT[SH::DVT1][SH::FC];
  if (a.rfold) {
    // the suffix of the later segments' local states (non-causal: the total),
    // summed in the scan's order (last segment first)
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) RT[dt][fc] = zero4();
    for (int q = a.segments - 1; q > (CAUSAL ? seg : -1); --q) {
      const float* in = a.rstate + ((size_t)bh * a.segments + q) * SH::STATE;
#pragma unroll
      for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc)
          RT[dt][fc] += *reinterpret_cast<const f32x4*>(in + state_off<SH>(w, dt, fc, l));
    }
  } else {
    const float* in = a.rstate + ((size_t)bh * a.segments + (CAUSAL ? seg : 0)) * SH::STATE;
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc)
        RT[dt][fc] = *reinterpret_cast<const f32x4*>(in + state_off<SH>(w, dt, fc, l));
  }
  // this wave's dW' partial starts from the query side's (dQ sweep) partial
  // of this workgroup position
  f32x4 DW[SH::PR][DT];
  {
    const size_t nmat = NS ? 2 : 1;
    const float* qpart = a.dwpart + (((size_t)0 * a.BH + bh) * a.segments + seg) * nmat * SH::M * D;
#pragma unroll
    for (int pr = 0; pr < SH::PR; ++pr)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        DW[pr][dt] = *reinterpret_cast<const f32x4*>(qpart + dw_tile_off<SH, D>(w, pr, dt, l));
  }
  float dtau_acc = 0.f;

  // dX fragments of this wave's d tiles w % DT (+ NW, ...)
  Frag<T> wf[DX_LDS ? 1 : NDK][DX_LDS ? 1 : NW][WTS::KP];
  if constexpr (DX_LDS) {
    for (int i = threadIdx.x; i < NW * NDX; i += SH::NT)
      DXL[i / NDX][i % NDX] = FragBlock<T, D, FW, NS>::dx(a.wfrag, h, NW, i / NDX)[i % NDX];
  } else {
#pragma unroll
    for (int kd = 0; kd < NDK; ++kd)
#pragma unroll
      for (int ww = 0; ww < NW; ++ww)
#pragma unroll
        for (int ks = 0; ks < WTS::KP; ++ks)
          wf[kd][ww][ks] = FragBlock<T, D, FW, NS>::dx(a.wfrag, h, NW, ww)[((w % DT + kd * NW) * WTS::KP + ks) * WAVE + l];
  }
  if (CAUSAL) {   // the zero tile of either intra-chunk matrix, and the zero row of -delta
    if (w < 2) {
      Frag<T> z;
      z.zero();
      if (w == 0) MP[1][l] = z;
      else AP[0][1][l] = AP[NSA - 1][1][l] = z;
    }
    for (int i = threadIdx.x; i < 2 * 3 * DLD; i += SH::NT) DLT2[i / (3 * DLD)][i % (3 * DLD)] = T(0.0f);
    __syncthreads();
  }
  // Store the prefetched rows into the buffers of sweep step i, which takes
  // the chunk at token tn, and prefetch the chunk before it (itself again when
  // it is the first: the prefetch is issued on every step, from an in-range chunk).
  auto stage = [&](int i, int cn) {
    const int par = i & 1, tn = cn * SH::CH;
    if (HALVES == 1 || half == 0) {
      st[0].store(XK2[par], SCK, [&](int t, auto ssq) {
        SSK2[par][t] = ssq;
        return row_scale(ssq, inv_c, a.s_const, tn + t < a.N);
      });
      if (CAUSAL) st[1].store(XQ, SCQ, [&](int t, auto ssq) { return row_scale(ssq, inv_c, a.s_const, tn + t < a.N); });
    }
    if (HALVES == 1 || half == 1) {
      st[SV].store(XV);
      if (CAUSAL) {
        st[SDO].store(XDO2[par]);
        const int t = StX::tid();
        if (t < SH::CH) {
          INV[t] = gs_next.x;
          DEL[t] = gs_next.y;
          float hi, lo;
          neg_split<T>(gs_next.y, hi, lo);
          DLT2[par][t] = (T)hi;
          DLT2[par][DLD + t] = (T)lo;
        }
      }
    }
    fetch((cn - 1 >= c0 ? cn - 1 : cn) * SH::CH);
  };
  // the bf16 copy of R' and the R' operand fragments of feature tile fc, from one conversion
  auto r_frags = [&](int fc, Frag<T> (&rp)[KG], bool store) {
#pragma unroll
    for (int kd = 0; kd < KG; ++kd) {
      rp[kd] = pair_tiles<T>(RT[2 * kd][fc], 2 * kd + 1 < SH::DVT1 ? RT[2 * kd + 1][fc] : zero4());
      if (store) {
        if (2 * kd + 1 < SH::DVT) {
          store_frag_nm<T>(RL[w], RLP, fc * 16, (2 * kd) * 16, (2 * kd + 1) * 16, rp[kd]);
        } else if (2 * kd < SH::DVT) {
          store_tile_nm<T>(RL[w], RLP, fc * 16, (2 * kd) * 16, RT[2 * kd][fc]);
        }
      }
    }
  };
  // One tile (query tile tq, key tile tk) of an intra-chunk matrix, masked to
  // keys at or before the query, into its half of the operand fragment.
  // (lo: its remainder's, or nullptr)
  auto store_intra = [&](Frag<T>* M, Frag<T>* lo, int tq, int tk, f32x4 v) {
    if (tq == tk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = 4 * g + i >= r ? v[i] : 0.f;
    }
    T* o = reinterpret_cast<T*>(&M[tk * WAVE + l]) + 4 * tq;
    T hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { hi[i] = (T)v[i]; o[i] = hi[i]; }
    if (lo) {
      T* ol = reinterpret_cast<T*>(&lo[tk * WAVE + l]) + 4 * tq;
#pragma unroll
      for (int i = 0; i < 4; ++i) ol[i] = (T)finite_low(v[i] - (float)hi[i]);
    }
  };
  // Projection fragments, reloaded per chunk (held for the whole sweep they
  // would not fit the registers).
  FreqSlice<T, D, FW, NS> fs;
  if (!CAUSAL) {   // one R' for every chunk
#pragma unroll
    for (int fc = 0; fc < SH::FC; ++fc) {
      Frag<T> rp[KG];
      r_frags(fc, rp, true);
    }
  }
  if (c0 < c1) {
    fs.load_frags(wproj);
    stage(0, c1 - 1);
  }
  __syncthreads();
  for (int c = c1 - 1; c >= c0; --c) {
    const int step = c1 - 1 - c;
    const int par = step & 1;
    IO* XK = XK2[par];
    IO* XDO = XDO2[CAUSAL ? par : 0];
    const T* DLT = DLT2[par];
    const int tok0 = c * SH::CH;
    const RowBuf dkb(dK, D, tok0, a.N, SH::CH), dvb(dV, SH::DV, tok0, a.N, SH::CH);

    // ---- interval 1
    // phi(Q)/den as [token][feature] in the wave's LDS block: read back as it is
    // for A, transposed for the token sums
    if (CAUSAL) {
#pragma unroll
      for (int tt = 0; tt < SH::TT; ++tt) {
        ProjT<T> p[SH::PR];
        float sc;
        project_tile_lds<T, D, FW, NS, StX::LD>(fs, XQ, SCQ, tt, p, sc);
        sc *= INV[tt * 16 + r];
#pragma unroll
        for (int ft = 0; ft < SH::FT; ++ft)
          PT[tt][w * SH::FT + ft].put(l, features<T, SH::FT, NS>(p, ft, sc, fv));
      }
    }
    // phi(K), with the factors of the chain rule kept in fp32: cos P1, sin P1,
    // s e cos P2 and s e sin P2 (stationary: s e alone)
    f32x4 kc[SH::FT][SH::TT], ks1[SH::FT][SH::TT], kw[SH::FT][SH::TT], kz[NS ? SH::FT : 1][SH::TT];
#pragma unroll
    for (int tt = 0; tt < SH::TT; ++tt) {
      ProjT<T> p[SH::PR];
      float sc;
      project_tile_lds<T, D, FW, NS, StX::LD>(fs, XK, SCK, tt, p, sc);
#pragma unroll
      for (int ft = 0; ft < SH::FT; ++ft) {
        Frag<T> f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float se = !MASK || ft * 16 + 4 * g + i < fv ? sc : 0.f;
          float s1, c1v;
          sincos_rev(p[ft][i], s1, c1v);
          float wv = se;
          if constexpr (NS) {
            float s2, c2;
            sincos_rev(p[SH::FT + ft][i], s2, c2);
            wv = se * c2;
            kz[ft][tt][i] = se * s2;
          }
          kc[ft][tt][i] = c1v;
          ks1[ft][tt][i] = s1;
          kw[ft][tt][i] = wv;
          f.set(i, c1v * wv);
          f.set(4 + i, s1 * wv);
        }
        PK[tt][w * SH::FT + ft][l] = f;
      }
    }
    // R' share of dphi(K)^T[feature][key] = R'^T-rows x [V | 1] + phi(Q)^T M
    f32x4 dph[SH::FC][SH::TT];
    {
      Frag<T> vf[SH::TT][KG];
#pragma unroll
      for (int tk = 0; tk < SH::TT; ++tk)
#pragma unroll
        for (int kd = 0; kd < KG; ++kd) {
          if (32 * kd < SH::DV) {
            vf[tk][kd] = lds_tok_frag<T>(reinterpret_cast<const T*>(XV) + (tk * 16 + r) * StV::LD, kd);
          } else {
            Frag<T> f;
            f.zero();
            if (g == 0) { f.set(0, 1.0f); f.set(1, 1.0f); }
            vf[tk][kd] = f;
          }
        }
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) {
        Frag<T> rp[KG];
        r_frags(fc, rp, CAUSAL);
#pragma unroll
        for (int tk = 0; tk < SH::TT; ++tk) {
          dph[fc][tk] = zero4();
#pragma unroll
          for (int kd = 0; kd < KG; ++kd) mma(dph[fc][tk], rp[kd], vf[tk][kd]);
        }
      }
    }
    // M tiles: the last three waves, one each
    if (CAUSAL && w >= NW - 3) {
      const int tq = w == NW - 1 ? 0 : 1, tk = w == NW - 3 ? 1 : 0;   // (0,0), (1,0), (1,1)
      f32x4 m = zero4();
#pragma unroll
      for (int kd = 0; kd < SH::DV / 32; ++kd) {
        Frag<T> ao, bv;
        lds_row8(ao, XDO + (tq * 16 + r) * StV::LD, kd * 32 + 8 * g);
        lds_row8(bv, XV + (tk * 16 + r) * StV::LD, kd * 32 + 8 * g);
        mma(m, ao, bv);
      }
      m -= *reinterpret_cast<const f32x4*>(DEL + tq * 16 + 4 * g);
      store_intra(&MP[0][0], nullptr, tq, tk, m);
    }
    __syncthreads();   // phi(Q), phi(K), R' and M complete; the rows of Q and V are read

    // ---- interval 2
    if constexpr (ACC && D == 64 && NW == 4 && NS && CAUSAL) {
      // also here where the old values of an earlier group leave too few registers (10
      // spilled, 7 so; B*H = 32, N = 2048, m = 192 training step 359 and 355 us)
      asm volatile("" : "+v"(l));
      r = l % 16;
      g = l / 16;
    }
    // an earlier group's dK and dV of this chunk (rows past N read zero)
    f32x4 old_k[ACC ? NOT : 1], old_v[ACC ? NOT : 1];
    if (ACC) {
#pragma unroll
      for (int k = 0; k < NOT; ++k) {
        const int ot = w + k * NW, off = ((ot / DT * 16 + r) * D + ot % DT * 16 + 4 * g) * 4;
        if (ot < DT * SH::TT) {
          old_k[k] = dkb.load_f4(off);
          old_v[k] = dvb.load_f4(off);
        }
      }
    }
    // A tiles: the first three waves, one each
    if (CAUSAL && w < 3) {
      const int tq = w == 0 ? 0 : 1, tk = w == 2 ? 1 : 0;
      f32x4 at = zero4();
#pragma unroll
      for (int ft = 0; ft < NFT; ++ft)
        mma(at, PT[tq][ft].get(l), PK[tk][ft][l]);
      store_intra(&AP[0][0][0], NSA == 2 ? &AP[1][0][0] : nullptr, tq, tk, at);
    }
    if (CAUSAL) {
      // M share of dphi(K), and R'^T += [dO | -delta]^T-rows x phi(Q)/den
      Frag<T> gt[SH::DVT1], mp[SH::TT];
#pragma unroll
      for (int tk = 0; tk < SH::TT; ++tk) mp[tk] = MP[tk][l];
#pragma unroll
      for (int dt = 0; dt < SH::DVT; ++dt) gt[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XDO), StV::LD, 4 * g, 16 + 4 * g, dt * 16);
      gt[SH::DVT] = lds_tok_frag<T>(DLT + (r < 2 ? r : 2) * DLD, 0);
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) {
        const Frag<T> pq = tr_of_frags(PT[0][w * SH::FT + fc / 2], PT[SH::TT - 1][w * SH::FT + fc / 2], fc % 2);
#pragma unroll
        for (int tk = 0; tk < SH::TT; ++tk) mma(dph[fc][tk], pq, mp[tk]);
#pragma unroll
        for (int dt = 0; dt < SH::DVT1; ++dt) mma(RT[dt][fc], gt[dt], pq);
      }
    }
    // R' share of this wave's dV^T tiles [value col][key] over all features
    f32x4 dv[NOT];
#pragma unroll
    for (int k = 0; k < NOT; ++k) dv[k] = zero4();
#pragma unroll
    for (int ft = 0; ft < NFT; ++ft)
#pragma unroll
      for (int k = 0; k < NOT; ++k) {
        const int ot = w + k * NW;
        if (DT * SH::TT % NW == 0 || ot < DT * SH::TT) {
          const Frag<T> rt = lds_tr_frag<T>(RL[ft / SH::FT], RLP, (2 * (ft % SH::FT)) * 16 + 4 * g,
                                            (2 * (ft % SH::FT) + 1) * 16 + 4 * g, ot % DT * 16);
          if constexpr (CAUSAL) mma_tree(dv[k], rt, PK[ot / DT][ft][l]);
          else mma(dv[k], rt, PK[ot / DT][ft][l]);
        }
      }
    // chain rule through phi(K): with t = cos P1 da + sin P1 db and
    // u = cos P1 db - sin P1 da, dP1 = s e cos P2 u, dP2 = -s e sin P2 t and
    // <phi, dphi> = s e cos P2 t; dP as [token][projection row] in LDS
#pragma unroll
    for (int tt = 0; tt < SH::TT; ++tt) {
      float gs = 0.f;
      f32x4 dp[SH::PR];
#pragma unroll
      for (int ft = 0; ft < SH::FT; ++ft) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float da = dph[2 * ft][tt][i], db = dph[2 * ft + 1][tt][i];
          const float t = kc[ft][tt][i] * da + ks1[ft][tt][i] * db;
          const float u = kc[ft][tt][i] * db - ks1[ft][tt][i] * da;
          dp[ft][i] = kw[ft][tt][i] * u;
          if constexpr (NS) dp[SH::FT + ft][i] = -kz[ft][tt][i] * t;
          gs += kw[ft][tt][i] * t;
        }
      }
#pragma unroll
      for (int ks = 0; ks < WTS::KP; ++ks)
        DP[tt][w * WTS::KP + ks].put(l, pair_tiles<T>(dp[2 * ks], 2 * ks + 1 < SH::PR ? dp[2 * ks + 1] : zero4()));
      gs = group_sum_swap(gs);
      if (g == 0) GP[tt * 16 + r][w] = gs;
    }
    // the next chunk's rows (the last step stages its own rows again, unused)
    stage(step + 1, c - 1 >= c0 ? c - 1 : c);
    __syncthreads();   // dP, g shares, A and the next chunk's rows complete

    // ---- interval 3
    // the lane index again, opaque: its uses from here to the next interval 3
    // compute their addresses once per chunk instead of holding each one in a
    // register for the whole sweep (they spilled)
    asm volatile("" : "+v"(l));
    r = l % 16;
    g = l / 16;
    fs.load_frags(wproj);   // the next chunk's (the last step's are unused)
    // dV: the A share; dK = dP W' over all projection rows + (2/c) g k, with
    // g = <phi(K), dphi(K)>; dtau -= g ||k||^2 / c
    f32x4 dk[NOT];
#pragma unroll
    for (int k = 0; k < NOT; ++k) {
      const int ot = w + k * NW, dt = ot % DT, tt = ot / DT;
      dk[k] = zero4();
      if (DT * SH::TT % NW != 0 && ot >= DT * SH::TT) continue;
      if (CAUSAL) {
        const Frag<T> gt = lds_tr_frag<T>(reinterpret_cast<const T*>(XDO), StV::LD, 4 * g, 16 + 4 * g, dt * 16);
#pragma unroll
        for (int p = 0; p < NSA; ++p) mma_tree(dv[k], gt, AP[p][tt][l]);
      }
#pragma unroll
      for (int ww = 0; ww < NW; ++ww)
#pragma unroll
        for (int ks = 0; ks < WTS::KP; ++ks) {
          const Frag<T> b = DP[tt][ww * WTS::KP + ks].get(l);
          if constexpr (DX_LDS) mma(dk[k], DXL[ww][(dt * WTS::KP + ks) * WAVE + l], b);
          else mma(dk[k], wf[k % NDK][ww][ks], b);
        }
    }
#pragma unroll
    for (int k = 0; k < NOT; ++k) {
      const int ot = w + k * NW, dt = ot % DT, tt = ot / DT;
      if (DT * SH::TT % NW != 0 && ot >= DT * SH::TT) continue;
      const int tl = tt * 16 + r, off = (tl * D + dt * 16 + 4 * g) * 4;
      if (ACC) dv[k] += old_v[k];   // later frequency groups add their share
      dvb.store_f4(off, dv[k]);
      float gg = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ww += 4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&GP[tl][ww]);
        gg += (v[0] + v[1]) + (v[2] + v[3]);
      }
      const float k2 = 2.0f * inv_c * gg;
      const IO* kr = XK + tl * StX::LD + dt * 16 + 4 * g;
#pragma unroll
      for (int i = 0; i < 4; ++i) dk[k][i] += k2 * io_to_float(kr[i]);
      if (ACC) dk[k] += old_k[k];
      dkb.store_f4(off, dk[k]);
      const float dt_term = gg * SSK2[par][tl] * inv_c;
      dtau_acc -= (dt == 0 && g == 0 && tok0 + tl < a.N) ? dt_term : 0.f;
    }
    {
      // one 32-token k-step per chunk
      Frag<T> xk[DT];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) xk[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XK), StX::LD, 4 * g, 16 + 4 * g, dt * 16);
#pragma unroll
      for (int pr = 0; pr < SH::PR; ++pr) {
        const Frag<T> dpt = tr_of_frags(DP[0][w * WTS::KP + pr / 2], DP[SH::TT - 1][w * WTS::KP + pr / 2], pr % 2);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) mma(DW[pr][dt], dpt, xk[dt]);
      }
    }
  }
  const size_t nmat = NS ? 2 : 1;
  float* out = a.dwpart + (((size_t)1 * a.BH + bh) * a.segments + seg) * nmat * SH::M * D;
  dump_dw<SH, D, FW, NS>(out, DW, w * FW);
  // dtau partial of this workgroup: fixed-order tree sum
  TRED[threadIdx.x] = dtau_acc;
  __syncthreads();
  for (int s = SH::NT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) TRED[threadIdx.x] += TRED[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.dtaupart[(size_t)bh * a.segments + seg] = TRED[0];
}

// ---------------------------------------------------------------------------
// Fixed-order reduction of the frequency-gradient and dtau partials.
// dwpart: [2][B*H][P][nmat][m][d]; the key side's blocks hold the sums of
// both sides in [matrix][m][d] order.  dW'1, dW'2 -> dW1 = (dW'1+dW'2)/2,
// dW2 = (dW'1-dW'2)/2 because W'1 = (W1+W2)/2 and W'2 = (W1-W2)/2.
// ---------------------------------------------------------------------------
template <int NMAT>
__global__ __launch_bounds__(256) void k_bwd_reduce(BwdArgs a, int md4, int d) {
  // 256 elements (f, k) of one head per workgroup, 4 consecutive per thread;
  // the 4 waves split the list of partials (b, segment; each already the sum
  // of the query and key sides) round-robin and
  // issue a batch of loads of every matrix before summing it (a partial past
  // the list reads the last one, added as zero), then the 4 wave sums are
  // combined in a fixed order.
  constexpr int BATCH = 8;
  __shared__ float4 part[NMAT][4][64];
  const int e4 = blockIdx.x * 64 + (threadIdx.x % 64);
  const int q = threadIdx.x / 64;
  const int h = blockIdx.y;
  const int count = a.B * a.segments;
  const float4* src = reinterpret_cast<const float4*>(a.dwpart);
  float4 acc[NMAT];
#pragma unroll
  for (int mat = 0; mat < NMAT; ++mat) acc[mat] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (e4 < md4) {
    for (int i0 = q; i0 < count; i0 += 4 * BATCH) {
      float4 v[BATCH][NMAT];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int j = min(i0 + 4 * u, count - 1);
        const int b = j / a.segments, p = j % a.segments;
        const size_t blk = ((size_t)1 * a.BH + (size_t)b * a.H + h) * a.segments + p;
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat) v[u][mat] = src[(blk * NMAT + mat) * md4 + e4];
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const float k = i0 + 4 * u < count ? 1.f : 0.f;
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat) {
          acc[mat].x += k * v[u][mat].x; acc[mat].y += k * v[u][mat].y;
          acc[mat].z += k * v[u][mat].z; acc[mat].w += k * v[u][mat].w;
        }
      }
    }
  }
#pragma unroll
  for (int mat = 0; mat < NMAT; ++mat) part[mat][q][threadIdx.x % 64] = acc[mat];
  __syncthreads();
  if (q == 0 && e4 < md4) {
    const int t = threadIdx.x;
    float4 x[NMAT];
#pragma unroll
    for (int mat = 0; mat < NMAT; ++mat) {
      const float4 p0 = part[mat][0][t], p1 = part[mat][1][t], p2 = part[mat][2][t], p3 = part[mat][3][t];
      x[mat] = make_float4((p0.x + p1.x) + (p2.x + p3.x), (p0.y + p1.y) + (p2.y + p3.y),
                           (p0.z + p1.z) + (p2.z + p3.z), (p0.w + p1.w) + (p2.w + p3.w));
    }
    float4* o1 = reinterpret_cast<float4*>(a.dW1 + (size_t)h * a.dw_stride) + e4;
    if (4 * e4 / d >= a.fvalid) {
      // a padding row of a last frequency group: no output row
    } else if (NMAT == 2) {
      float4* o2 = reinterpret_cast<float4*>(a.dW2 + (size_t)h * a.dw_stride) + e4;
      const float4 u = x[0], w = x[NMAT - 1];
      *o1 = make_float4(0.5f * (u.x + w.x), 0.5f * (u.y + w.y), 0.5f * (u.z + w.z), 0.5f * (u.w + w.w));
      *o2 = make_float4(0.5f * (u.x - w.x), 0.5f * (u.y - w.y), 0.5f * (u.z - w.z), 0.5f * (u.w - w.w));
    } else {
      *o1 = x[0];
    }
  }
  if (a.dtau && blockIdx.x == 0 && q == 1) {
    // one wave, every lane its share of the partials in order, then a fixed tree
    float s = 0.f;
    for (int j = threadIdx.x % 64; j < count; j += 64)
      s += a.dtaupart[((size_t)(j / a.segments) * a.H + h) * a.segments + j % a.segments];
    s = group_sum(lane_sum<16>(s));
    if (threadIdx.x % 64 == 0) a.dtau[h] = a.acc ? a.dtau[h] + s : s;
  }
}

// ---------------------------------------------------------------------------
// Host-side dispatch.
// ---------------------------------------------------------------------------
// FW frequencies per wave, NW waves per workgroup, in every kernel.
template <class T, int D, bool NS, int FW, int NW>
static hipError_t run_bwd_t(const BwdArgs& a, bool causal, hipStream_t st) {
  typedef Shape<T, D, FW, NW, NS, BWD_CHUNK> SH;
  const dim3 grid(a.segments * a.BH);
  k_prep_freqs<T, D, FW, NW, NS><<<dim3(a.H, NW, 2), WAVE, 0, st>>>(a.W1, a.W2, a.wfrag, a.w_stride);
  // With the forward's key-side states passed in, the dQ sweep does the
  // pre-pass's query-side work itself and no pre-pass runs; the R' local
  // states it leaves feed the scan, or the dK/dV sweep's own suffix sum.
  const bool wr = a.fstate != nullptr;
  // a padded frequency group (it runs first, so it never adds) takes the
  // masking kernel variants
  const bool masked = a.fvalid < SH::M;
  constexpr bool CAN_MASK = group_can_pad(D, SH::M);
  if (masked && (!CAN_MASK || a.acc)) return hipErrorInvalidValue;
  auto scan_r = [&]() -> hipError_t {
    if (a.rfold) return hipSuccess;
    return launch_state_scan(wr ? nullptr : a.sstate, a.rstate, a.BH, a.segments, 1, SH::STATE, causal, st,
                             a.segments);
  };
  if (!wr) {
    timing_mark(KC_BWD_PREPASS, st, true);
    if constexpr (CAN_MASK) {
      if (masked) k_bwd_prepass<T, D, FW, NW, NS, true><<<grid, SH::NT, 0, st>>>(a);
    }
    if (!masked) k_bwd_prepass<T, D, FW, NW, NS><<<grid, SH::NT, 0, st>>>(a);
    timing_mark(KC_BWD_PREPASS, st, false);
    const hipError_t e = scan_r();
    if (e != hipSuccess) return e;
  }
  timing_mark(KC_BWD_DQ, st, true);
  // a later frequency group adds into the earlier groups' outputs
  {
    const hipError_t e = launch_bwd_dq<T, D, FW, NW, NS>(a, causal, a.acc != 0, wr, masked, st);
    if (e != hipSuccess) return e;
  }
  timing_mark(KC_BWD_DQ, st, false);
  if (wr) {
    const hipError_t e = scan_r();
    if (e != hipSuccess) return e;
  }
  timing_mark(KC_BWD_DKV, st, true);
  if (a.acc) {
    if (causal)
      k_bwd_dkv<T, D, FW, NW, NS, true, true><<<grid, SH::NT, 0, st>>>(a);
    else
      k_bwd_dkv<T, D, FW, NW, NS, false, true><<<grid, SH::NT, 0, st>>>(a);
  } else if (masked) {
    if constexpr (CAN_MASK) {
      if (causal)
        k_bwd_dkv<T, D, FW, NW, NS, true, false, true><<<grid, SH::NT, 0, st>>>(a);
      else
        k_bwd_dkv<T, D, FW, NW, NS, false, false, true><<<grid, SH::NT, 0, st>>>(a);
    }
  } else {
    if (causal)
      k_bwd_dkv<T, D, FW, NW, NS, true, false><<<grid, SH::NT, 0, st>>>(a);
    else
      k_bwd_dkv<T, D, FW, NW, NS, false, false><<<grid, SH::NT, 0, st>>>(a);
  }
  timing_mark(KC_BWD_DKV, st, false);
  static_assert((SH::M * D) % 4 == 0, "the reduce moves 4 floats per thread");
  constexpr int MD4 = SH::M * D / 4;
  dim3 rgrid((MD4 + 63) / 64, a.H);
  timing_mark(KC_BWD_REDUCE, st, true);
  k_bwd_reduce<NS ? 2 : 1><<<rgrid, 256, 0, st>>>(a, MD4, D);
  timing_mark(KC_BWD_REDUCE, st, false);
  return hipGetLastError();
}

template <class T, int D, int FW, int NW>
static hipError_t run_bwd_v(const BwdArgs& a, bool ns, bool causal, hipStream_t st) {
  return ns ? run_bwd_t<T, D, true, FW, NW>(a, causal, st)
            : run_bwd_t<T, D, false, FW, NW>(a, causal, st);
}

hipError_t launch_bwd(const BwdArgs& a, const KernelShape& ks, hipStream_t st) {
  if (ks.bf16) {
    if (ks.d == 32 && ks.m == 64) return run_bwd_v<__bf16, 32, 16, 4>(a, ks.nonstationary, ks.causal, st);
    if (ks.d == 32 && ks.m == 128) return run_bwd_v<__bf16, 32, 16, 8>(a, ks.nonstationary, ks.causal, st);
    if (ks.d == 64 && ks.m == 64) return run_bwd_v<__bf16, 64, 16, 4>(a, ks.nonstationary, ks.causal, st);
    if (ks.d == 64 && ks.m == 128) return run_bwd_v<__bf16, 64, 16, 8>(a, ks.nonstationary, ks.causal, st);
    if (ks.d == 128 && ks.m == 64) return run_bwd_v<__bf16, 128, 16, 4>(a, ks.nonstationary, ks.causal, st);
  } else {
    if (ks.d == 32 && ks.m == 64) return run_bwd_v<float, 32, 16, 4>(a, ks.nonstationary, ks.causal, st);
  }
  return hipErrorNotSupported;
}

size_t bwd_state_floats(const KernelShape& ks) { return fwd_state_floats(ks); }
// both sides (query rows and key rows) of the frequency-gradient partials
size_t bwd_dw_floats(const KernelShape& ks) {
  return (size_t)2 * (ks.nonstationary ? 2 : 1) * ks.m * ks.d;
}

}  // namespace flex
