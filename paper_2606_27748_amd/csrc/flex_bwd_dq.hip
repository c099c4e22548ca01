// dQ sweep of the RFF linear attention backward (the derivation and the
// kernel list are in flex_bwd.hip).  A translation unit of its own, so that
// it can be compiled with MFMA results placed in VGPRs, which suits this
// sweep (its results mostly feed vector code) but not the others.
#include "flex_bwd_common.hpp"

namespace flex {

// ---------------------------------------------------------------------------
// dQ: ascending sweep with the key-side prefix state S'.
//
// A chunk has three intervals between two barriers, as in the dK/dV sweep:
//   1  (waves split the frequencies) phi(K) and phi(Q)/den; the S' share of
//      dphi(Q); three waves form the tiles of M^T, M = dO V^T - delta
//   2  (frequencies) the M share of dphi(Q), the S' (and R') update, the chain
//      rule, dP to LDS, the next chunk's rows to LDS
//   3  (output tiles) dQ = dP W'; (frequencies) dW' += dP^T Q
// us per pass before (every wave forming all of M^T, a barrier of its own for
// the rows, K and V staged without need in the non-causal sweep) and after:
// training step d = 64, m = 128 (B*H = 32, N = 8192) 424 and 411, d = 128,
// m = 256 2439 and 2427, encoder training (non-causal m = 64) 232 and 227.
// ---------------------------------------------------------------------------
// ACC: add dQ to the values an earlier frequency group stored (loaded ahead of
// the next chunk's prefetch).
// WR: this sweep also does the pre-pass's query-side work (used when the
// forward's key-side states are passed in, so no pre-pass runs): the per-token
// 1/den and delta = dO . O, from the staging registers, written for the dK/dV
// sweep, and the segment-local R'^T = sum [dO | -delta]^T-rows x phi(Q)/den.
template <class T, int D, int FW, int NW, bool NS, bool CAUSAL, bool ACC, bool WR, bool MASK = false>
__global__ __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(bwd_waves_per_eu(IsBf16<T>::value, D))))
void k_bwd_dq(BwdArgs a) {
  typedef Shape<T, D, FW, NW, NS, BWD_CHUNK> SH;
  typedef typename Io<T>::type IO;
  // With at least two threads per 16-byte vector of a chunk's rows, half of the
  // waves stage Q, K and V and the other half dO and O.
  constexpr int HALVES = 2 * SH::CH * D * (int)sizeof(IO) / 16 <= SH::NT ? 2 : 1;
  constexpr int NTH = SH::NT / HALVES;
  typedef RowStage<IO, D, NTH, SH::CH> StX;
  static_assert(D == SH::DV && (StX::NV % NTH == 0 || StX::NV < NTH), "one stage type, the same row vectors per thread");
  typedef WTSlice<T, D, FW, NS> WTS;
  constexpr int DT = D / 16;
  constexpr int KG = (SH::DVT1 + 1) / 2;        // k-steps over [dO | -delta]
  constexpr int NOT = (DT * SH::TT + NW - 1) / NW;   // dQ tiles per wave (at most)
  constexpr int NDX = FragBlock<T, D, FW, NS>::NT_ * WAVE;   // dX fragments per wave
  static_assert(SH::TT == 2 && SH::KT == 1 && SH::FT == 1 && NW >= 4, "32-token chunks, three waves for the intra-chunk tiles");
  // rows read in interval 1 only (K) need one staging buffer (stored in
  // interval 2), the others two, by chunk parity
  __shared__ __attribute__((aligned(16))) IO XQ2[2][StX::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XK[CAUSAL ? StX::LDS_ELEMS : 8];
  __shared__ __attribute__((aligned(16))) IO XV2[CAUSAL ? 2 : 1][CAUSAL ? StX::LDS_ELEMS : 8];
  __shared__ __attribute__((aligned(16))) IO XDO2[2][StX::LDS_ELEMS];
  // phi(Q)/den, then dP, operand fragments (dP: k = pairs of projection row tiles)
  __shared__ FragLds<T> DP[SH::TT][NW];
  __shared__ Frag<T> MT[CAUSAL ? SH::TT : 1][WAVE];   // M^T: [query tile], k = key tokens
  // dW' partial: in registers, except at d = 64 causal, where the two states
  // take them
  constexpr bool DW_REG = D != 64 || !CAUSAL;
  __shared__ __attribute__((aligned(16))) float DWL[DW_REG ? 1 : NW][DW_REG ? 4 : SH::PR * DT * WAVE * 4];
  // dX fragments of every wave's projection rows: held in registers with four
  // waves (each then has DT / 4 d tiles), in LDS with eight
  constexpr bool DX_LDS = NW > 4;
  constexpr int NDK = DT > NW ? DT / NW : 1;     // d tiles of one wave
  static_assert(DT <= NW ? NW % DT == 0 : DT % NW == 0, "a wave keeps its d tiles");
  __shared__ Frag<T> DXL[DX_LDS ? NW : 1][DX_LDS ? NDX : 1];
  __shared__ __attribute__((aligned(16))) float SCQ[SH::CH], SCK[SH::CH], INV[SH::CH], DEL[SH::CH];
  __shared__ __attribute__((aligned(16))) T DHL[SH::CH][2];   // -delta as a (hi, lo) pair
  constexpr int DLD = SH::CH + 8;
  __shared__ __attribute__((aligned(16))) T DLT2[2][3 * DLD];   // the same as operand rows, and a row of zeros

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
  const IO* Ob = static_cast<const IO*>(a.O) + (size_t)bh * a.N * SH::DV;
  const float* den = a.den + (size_t)bh * a.N;
  float* gst = a.gstats + (size_t)bh * a.N * 2;
  float* dQ = a.dQ + (size_t)bh * a.N * D;

  // stages: Q, K, V of the first half in st[0..2]; dO and O here (K and V only
  // for the intra-chunk terms of the causal sweep)
  const int half = HALVES == 2 ? w / (NW / 2) : 0;
  constexpr int SDO = HALVES == 2 ? 0 : 3, SO = SDO + 1;
  StX st[HALVES == 2 ? 3 : 5];
  constexpr int WPER = WR ? StX::PER : 1;
  float dn_next[WPER];
  float2 gs_next = make_float2(0.f, 0.f);
#pragma unroll
  for (int i = 0; i < WPER; ++i) dn_next[i] = 0.f;
  auto fetch = [&](int t0) {
    st[0].fetch(HALVES == 2 && half ? dO : Q, t0, a.N);
    // (two halves: a stage that this half does not use has a window of no rows,
    // whose loads read nothing and need no branch; with loads of other rows in their
    // place the training step d = 64, m = 128, B*H = 32, N = 8192 takes 406 us, so 403)
    if (CAUSAL || (WR && HALVES == 2))
      st[1].fetch(HALVES == 2 && half ? Ob : K, t0, HALVES == 1 || (half ? WR : CAUSAL) ? a.N : t0);
    if (CAUSAL) st[2].fetch(V, t0, HALVES == 2 && half ? t0 : a.N);
    if (HALVES == 1) {
      st[SDO].fetch(dO, t0, a.N);
      if (WR) st[SO].fetch(Ob, t0, a.N);
    }
    if (WR) {   // den of this thread's rows (rows past N read zero, unused)
      const RowBuf b(den, 1, t0, a.N, SH::CH);
#pragma unroll
      for (int i = 0; i < WPER; ++i) dn_next[i] = b.load_f1((StX::tid() + i * NTH) / StX::VPR * 4);
    } else {
      gs_next = load_gs(gst, t0, a.N, SH::CH, StX::tid());
    }
  };
  if (c0 < c1) fetch(c0 * SH::CH);
  const Frag<T>* wproj = FragBlock<T, D, FW, NS>::proj(a.wfrag, h, NW, w);
  const auto inv_c = inv_c_of<T>(a.tau[h]);

  f32x4 ST[SH::DVT1][SH::FC];
  if (a.fstate && a.ffold) {
    // the forward ran no scan: the exclusive prefix (total) of its local states,
    // summed in the scan's order (the same sum the forward sweep formed)
    const float* blk = a.fstate + (size_t)bh * a.segments * a.fsub * a.fstride;
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) ST[dt][fc] = zero4();
    for (int k = 0; k < (CAUSAL ? seg : a.segments) * a.fsub; ++k) {
      const float* in = blk + (size_t)k * a.fstride;
#pragma unroll
      for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc) ST[dt][fc] += fwd_state_tile_t<SH>(in, w, dt, fc);
    }
  } else if (a.fstate) {
    const float* in = a.fstate + ((size_t)bh * a.segments * a.fsub + (CAUSAL ? seg * a.fsub : 0)) * a.fstride;
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) ST[dt][fc] = fwd_state_tile_t<SH>(in, w, dt, fc);
  } else {
    const float* in = a.sstate + ((size_t)bh * a.segments + (CAUSAL ? seg : 0)) * SH::STATE;
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc)
        ST[dt][fc] = *reinterpret_cast<const f32x4*>(in + state_off<SH>(w, dt, fc, l));
  }
  f32x4 DW[DW_REG ? SH::PR : 1][DW_REG ? DT : 1];
  if constexpr (DW_REG) {
#pragma unroll
    for (int pr = 0; pr < SH::PR; ++pr)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) DW[pr][dt] = zero4();
  } else {
    for (int i = l; i < SH::PR * DT * WAVE; i += WAVE) *reinterpret_cast<f32x4*>(&DWL[w][i * 4]) = zero4();
  }
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
  // the zero tile of M^T, and the zero row of -delta
  if (CAUSAL && w == 0) {
    Frag<T> z;
    z.zero();
    MT[0][l] = z;
  }
  if (WR) for (int i = threadIdx.x; i < 2 * 3 * DLD; i += SH::NT) DLT2[i / (3 * DLD)][i % (3 * DLD)] = T(0.0f);
  __syncthreads();
  const Frag<T> ones = ones_col01<T>();
  f32x4 RT[WR ? SH::DVT1 : 1][WR ? SH::FC : 1];
#pragma unroll
  for (int dt = 0; dt < (WR ? SH::DVT1 : 1); ++dt)
#pragma unroll
    for (int fc = 0; fc < (WR ? SH::FC : 1); ++fc) RT[dt][fc] = zero4();

  // Store the prefetched rows of chunk cn into the buffers of sweep step i
  // and prefetch the next chunk (itself again when it is the last: the
  // prefetch is issued on every step, from an in-range chunk).
  auto put_delta = [&](int par, int t, float inv, float dl) {
    INV[t] = inv;
    DEL[t] = dl;
    float hi, lo;
    neg_split<T>(dl, hi, lo);
    DHL[t][0] = (T)hi;
    DHL[t][1] = (T)lo;
    if (WR) {
      DLT2[par][t] = (T)hi;
      DLT2[par][DLD + t] = (T)lo;
    }
  };
  auto stage = [&](int i, int cn) {
    const int par = i & 1, tn = cn * SH::CH;
    auto scale = [&](int t, auto ssq) { return row_scale(ssq, inv_c, a.s_const, tn + t < a.N); };
    if (HALVES == 1 || half == 0) {
      st[0].store(XQ2[par], SCQ, scale);
      if (CAUSAL) {
        st[1].store(XK, SCK, scale);
        st[2].store(XV2[par]);
      }
    }
    if (HALVES == 1 || half == 1) {
      st[SDO].store(XDO2[par]);
      if constexpr (WR) {
        // 1/den and delta of this thread's rows (rows past N: zero vectors, delta 0,
        // and their stores to memory are dropped)
        const RowBuf gb(gst, 2, tn, a.N, SH::CH);
#pragma unroll
        for (int k = 0; k < WPER; ++k) {
          const int v = StX::tid() + k * NTH, t = v / StX::VPR;
          float dsum = 0.f;
          const uint4 x = st[SDO].vec(k), y = st[SO].vec(k);
          const IO* ex = reinterpret_cast<const IO*>(&x);
          const IO* ey = reinterpret_cast<const IO*>(&y);
#pragma unroll
          for (int j = 0; j < StX::VEC; ++j) dsum += io_to_float(ex[j]) * io_to_float(ey[j]);
          dsum = lane_sum<StX::VPR>(dsum);
          const float rcp = 1.0f / dn_next[k];
          const float inv = tn + t < a.N ? rcp : 0.f;
          if (v < StX::NV && v % StX::VPR == 0) {
            put_delta(par, t, inv, dsum);
            gb.store_f2(t * 8, make_float2(inv, dsum));
          }
        }
      } else {
        if (StX::tid() < SH::CH) put_delta(par, StX::tid(), gs_next.x, gs_next.y);
      }
    }
    fetch((cn + 1 < c1 ? cn + 1 : cn) * SH::CH);
  };
  // projection fragments, reloaded per chunk (held for the whole sweep they
  // would not fit the registers)
  FreqSlice<T, D, FW, NS> fs;
  if (c0 < c1) {
    fs.load_frags(wproj);
    stage(0, c0);
  }
  __syncthreads();
  for (int c = c0; c < c1; ++c) {
    const int step = c - c0;
    const int par = step & 1;
    IO* XQ = XQ2[par];
    IO* XV = XV2[CAUSAL ? par : 0];
    IO* XDO = XDO2[par];
    const T* DLT = DLT2[par];
    const int tok0 = c * SH::CH;
    const RowBuf dqb(dQ, D, tok0, a.N, SH::CH);

    // ---- interval 1
    // phi(K) of this wave's features enters only contractions over the key
    // tokens: token-row fragments (k = tokens), no transpose
    Frag<T> pk[SH::FC];
    if (CAUSAL) feature_frags_rows<T, D, FW, NS, StX::LD>(fs, XK, SCK, 0, pk, fv);
    // phi(Q)/den, and the factors of the chain rule in fp32: cos P1, sin P1,
    // s e cos P2 / den and s e sin P2 / den (stationary: s e / den alone; the
    // 1/den of dphi(Q) is carried by these: the products are the same)
    f32x4 qc[SH::TT], qs[SH::TT], qw[SH::TT], qz[NS ? SH::TT : 1];
    Frag<T> phq[SH::TT];
#pragma unroll
    for (int tt = 0; tt < SH::TT; ++tt) {
      ProjT<T> p[SH::PR];
      float sc;
      project_tile_lds<T, D, FW, NS, StX::LD>(fs, XQ, SCQ, tt, p, sc);
      sc *= INV[tt * 16 + r];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float se = !MASK || 4 * g + i < fv ? sc : 0.f;
        float s1, c1v;
        sincos_rev(p[0][i], s1, c1v);
        float wv = se;
        if constexpr (NS) {
          float s2, c2;
          sincos_rev(p[1][i], s2, c2);
          wv = se * c2;
          qz[tt][i] = se * s2;
        }
        qc[tt][i] = c1v;
        qs[tt][i] = s1;
        qw[tt][i] = wv;
        if (WR) {
          phq[tt].set(i, c1v * wv);
          phq[tt].set(4 + i, s1 * wv);
        }
      }
    }
    // S' share of den * dphi(Q)^T[feature][query] = S'^T-rows x [dO | -delta] + phi(K)^T M^T
    f32x4 dph[SH::FC][SH::TT];
    {
      Frag<T> gf[SH::TT][KG];
#pragma unroll
      for (int tq = 0; tq < SH::TT; ++tq)
#pragma unroll
        for (int kd = 0; kd < KG; ++kd) {
          if (32 * kd < SH::DV) {
            gf[tq][kd] = lds_tok_frag<T>(reinterpret_cast<const T*>(XDO) + (tq * 16 + r) * StX::LD, kd);
          } else {
            Frag<T> f;
            f.zero();
            const T hi = DHL[tq * 16 + r][0], lo = DHL[tq * 16 + r][1];
            if (g == 0) { f.v[0] = hi; f.v[1] = lo; }
            gf[tq][kd] = f;
          }
        }
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
        for (int kd = 0; kd < KG; ++kd) {
          const Frag<T> sp = pair_tiles<T>(ST[2 * kd][fc], 2 * kd + 1 < SH::DVT1 ? ST[2 * kd + 1][fc] : zero4());
#pragma unroll
          for (int tq = 0; tq < SH::TT; ++tq) {
            if (kd == 0) dph[fc][tq] = zero4();
            mma(dph[fc][tq], sp, gf[tq][kd]);
          }
        }
    }
    // M^T tiles, rows = key tokens, cols = query tokens, keys at or before the
    // query: the last three waves, one each
    if (CAUSAL && w >= NW - 3) {
      const int tk = w == NW - 3 ? 1 : 0, tq = w == NW - 1 ? 0 : 1;   // (0,0), (0,1), (1,1)
      f32x4 m = zero4();
#pragma unroll
      for (int kd = 0; kd < SH::DV / 32; ++kd) {
        Frag<T> av, bo;
        lds_row8(av, XV + (tk * 16 + r) * StX::LD, kd * 32 + 8 * g);
        lds_row8(bo, XDO + (tq * 16 + r) * StX::LD, kd * 32 + 8 * g);
        mma(m, av, bo);
      }
      const float dl = DEL[tq * 16 + r];
      T* o = reinterpret_cast<T*>(&MT[CAUSAL ? tq : 0][l]) + 4 * tk;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float md = m[i] - dl;
        o[i] = (T)(tk < tq || 4 * g + i <= r ? md : 0.f);
      }
    }
    __syncthreads();   // M^T complete; K's rows are read, and the previous chunk's dP

    // ---- interval 2
    // an earlier group's dQ of this chunk (rows past N read zero)
    f32x4 old_q[ACC ? NOT : 1];
    if (ACC) {
#pragma unroll
      for (int k = 0; k < NOT; ++k) {
        const int ot = w + k * NW;
        if (ot < DT * SH::TT) old_q[k] = dqb.load_f4(((ot / DT * 16 + r) * D + ot % DT * 16 + 4 * g) * 4);
      }
    }
    if constexpr (WR) {
      // R'^T += [dO | -delta]^T-rows x phi(Q)/den, with phi(Q)/den read back
      // transposed from this wave's fragments (which take its dP after that)
#pragma unroll
      for (int tt = 0; tt < SH::TT; ++tt) DP[tt][w].put(l, phq[tt]);
      Frag<T> gt[SH::DVT1];
#pragma unroll
      for (int dt = 0; dt < SH::DVT; ++dt) gt[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XDO), StX::LD, 4 * g, 16 + 4 * g, dt * 16);
      gt[SH::DVT] = lds_tok_frag<T>(DLT + (r < 2 ? r : 2) * DLD, 0);
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) {
        const Frag<T> pq = tr_of_frags(DP[0][w], DP[1][w], fc);
#pragma unroll
        for (int dt = 0; dt < SH::DVT1; ++dt) mma(RT[dt][fc], gt[dt], pq);
      }
    }
    if (CAUSAL) {
      // M share of dphi(Q); S'^T += [V | 1]^T-rows x phi(K)
#pragma unroll
      for (int tq = 0; tq < SH::TT; ++tq) {
        const Frag<T> mt = MT[CAUSAL ? tq : 0][l];
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc) mma(dph[fc][tq], pk[fc], mt);
      }
#pragma unroll
      for (int dt = 0; dt < SH::DVT1; ++dt) {
        const Frag<T> vt = dt < SH::DVT ? lds_tr_frag<T>(reinterpret_cast<const T*>(XV), StX::LD, 4 * g, 16 + 4 * g, dt * 16) : ones;
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc) mma(ST[dt][fc], vt, pk[fc]);
      }
    }
    // chain rule through phi(Q) (as for K in the dK/dV sweep): dP per radian
#pragma unroll
    for (int tt = 0; tt < SH::TT; ++tt) {
      f32x4 d1, d2 = zero4();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float da = dph[0][tt][i], db = dph[1][tt][i];
        d1[i] = qw[tt][i] * (qc[tt][i] * db - qs[tt][i] * da);
        if constexpr (NS) d2[i] = -qz[tt][i] * (qc[tt][i] * da + qs[tt][i] * db);
      }
      DP[tt][w].put(l, pair_tiles<T>(d1, d2));
    }
    // the next chunk's rows (the last step stages its own rows again, unused)
    stage(step + 1, c + 1 < c1 ? c + 1 : c);
    __syncthreads();   // dP and the next chunk's rows complete

    // ---- interval 3
    // the lane index again, opaque: its uses from here to the next interval 3
    // compute their addresses once per chunk instead of holding each one in a
    // register for the whole sweep
    asm volatile("" : "+v"(l));
    r = l % 16;
    g = l / 16;
    fs.load_frags(wproj);   // the next chunk's (the last step's are unused)
    // dQ = dP W' over all projection rows, whole output tiles
    f32x4 acc[NOT];
#pragma unroll
    for (int k = 0; k < NOT; ++k) {
      const int ot = w + k * NW, dt = ot % DT, tt = ot / DT;
      acc[k] = zero4();
      if (DT * SH::TT % NW != 0 && ot >= DT * SH::TT) continue;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww)
#pragma unroll
        for (int ks = 0; ks < WTS::KP; ++ks) {
          if constexpr (DX_LDS) mma(acc[k], DXL[ww][(dt * WTS::KP + ks) * WAVE + l], DP[tt][ww].get(l));
          else mma(acc[k], wf[k % NDK][ww][ks], DP[tt][ww].get(l));
        }
    }
#pragma unroll
    for (int k = 0; k < NOT; ++k) {
      const int ot = w + k * NW, dt = ot % DT, tt = ot / DT;
      if (DT * SH::TT % NW != 0 && ot >= DT * SH::TT) continue;
      if (ACC) acc[k] += old_q[k];   // later frequency groups add their share
      dqb.store_f4(((tt * 16 + r) * D + dt * 16 + 4 * g) * 4, acc[k]);
    }
    // frequency gradient partial: dW'[rows][d] += dP^T Q, one 32-token k-step
    {
      Frag<T> xq[DT];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) xq[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XQ), StX::LD, 4 * g, 16 + 4 * g, dt * 16);
#pragma unroll
      for (int pr = 0; pr < SH::PR; ++pr) {
        const Frag<T> dpt = tr_of_frags(DP[0][w], DP[1][w], pr);
        if constexpr (DW_REG) {
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) mma(DW[pr][dt], dpt, xq[dt]);
        } else {
          dw_mma_row<D, T>(DWL[w], pr, dpt, xq);
        }
      }
    }
  }
  const size_t nmat = NS ? 2 : 1;
  float* out = a.dwpart + (((size_t)0 * a.BH + bh) * a.segments + seg) * nmat * SH::M * D;
#pragma unroll
  for (int pr = 0; pr < SH::PR; ++pr)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      f32x4 v;
      if constexpr (DW_REG) v = DW[pr][dt];
      else v = *reinterpret_cast<const f32x4*>(&DWL[w][((pr * DT + dt) * WAVE + l) * 4]);
      *reinterpret_cast<f32x4*>(out + dw_tile_off<SH, D>(w, pr, dt, l)) = v;
    }
  if constexpr (WR) {
    float* ro = a.rstate + ((size_t)bh * a.segments + seg) * SH::STATE;
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) *reinterpret_cast<f32x4*>(ro + state_off<SH>(w, dt, fc, l)) = RT[dt][fc];
  }
}

// Launch of the dQ sweep for one shape: grouped_acc adds into an earlier
// frequency group's dQ; wr does the pre-pass's query-side work
// (with the forward's key-side states).
template <class T, int D, int FW, int NW, bool NS, bool ACC, bool MASK>
static void launch_dq_acc(const BwdArgs& a, bool causal, bool wr, const dim3& grid, int nt, hipStream_t st) {
  if (wr) {
    if (causal) k_bwd_dq<T, D, FW, NW, NS, true, ACC, true, MASK><<<grid, nt, 0, st>>>(a);
    else k_bwd_dq<T, D, FW, NW, NS, false, ACC, true, MASK><<<grid, nt, 0, st>>>(a);
  } else {
    if (causal) k_bwd_dq<T, D, FW, NW, NS, true, ACC, false, MASK><<<grid, nt, 0, st>>>(a);
    else k_bwd_dq<T, D, FW, NW, NS, false, ACC, false, MASK><<<grid, nt, 0, st>>>(a);
  }
}

template <class T, int D, int FW, int NW, bool NS>
hipError_t launch_bwd_dq(const BwdArgs& a, bool causal, bool grouped_acc, bool wr, bool masked, hipStream_t st) {
  typedef Shape<T, D, FW, NW, NS, BWD_CHUNK> SA;
  const dim3 grid(a.segments * a.BH);
  if (masked) {   // a padded group: never adding
    if constexpr (group_can_pad(D, FW * NW)) {
      if (!grouped_acc) {
        launch_dq_acc<T, D, FW, NW, NS, false, true>(a, causal, wr, grid, SA::NT, st);
        return hipGetLastError();
      }
    }
    return hipErrorInvalidValue;
  }
  if (grouped_acc)
    launch_dq_acc<T, D, FW, NW, NS, true, false>(a, causal, wr, grid, SA::NT, st);
  else
    launch_dq_acc<T, D, FW, NW, NS, false, false>(a, causal, wr, grid, SA::NT, st);
  return hipGetLastError();
}

#define FLEX_DQ_SHAPE(T, D, FW, NW)                                                                  \
  template hipError_t launch_bwd_dq<T, D, FW, NW, true>(const BwdArgs&, bool, bool, bool, bool, hipStream_t); \
  template hipError_t launch_bwd_dq<T, D, FW, NW, false>(const BwdArgs&, bool, bool, bool, bool, hipStream_t);
FLEX_DQ_SHAPE(__bf16, 32, 16, 4)
FLEX_DQ_SHAPE(__bf16, 32, 16, 8)
FLEX_DQ_SHAPE(__bf16, 64, 16, 4)
FLEX_DQ_SHAPE(__bf16, 64, 16, 8)
FLEX_DQ_SHAPE(__bf16, 128, 16, 4)
FLEX_DQ_SHAPE(float, 32, 16, 4)
#undef FLEX_DQ_SHAPE

}  // namespace flex
