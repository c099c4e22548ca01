// Forward kernels of the RFF linear attention (Eq.(linear att), Sec. 2.2) with
// the Flexformer feature maps (Eq.(phi_n) / Eq.(phi_non), Sec. 3.1-3.2).
//
// Work decomposition.  A workgroup owns one (b,h) slice and one contiguous
// segment of 64-token chunks.  Its NW waves split the m frequencies: wave w
// owns frequencies [w*FW, (w+1)*FW), i.e. 2*FW of the d' = 2m features, and
// keeps its rows of the state S' = sum_j phi(K_j) [V_j ; 1]^T (d' x (dv+1),
// fp32) as MFMA accumulators.  Per chunk a wave forms phi(Q), phi(K) for its
// features on chip (projection + fused trig, never written to memory); the
// sweep hands them and the state to the other waves as operand fragments in
// LDS, and each wave then reads out whole output tiles over all features.
//
// Causal sequences are split into segments for occupancy:
//   k_fwd_state  : segment-local states (one pass over K, V),
//   k_state_scan : exclusive prefix over segments (causal) or the total
//                  (non-causal), fixed order, deterministic,
//   k_fwd_sweep  : per segment, carry-in state + chunk sweep, writes O, den.
#include "flex_common.hpp"
#include "flex_kernels.hpp"
#include "flex_stage.hpp"

namespace flex {

// ---------------------------------------------------------------------------
// Segment-local state: S'_seg = sum over the segment's tokens of phi(K)[V;1]^T.
// ---------------------------------------------------------------------------
// MASK: the variant for a padded frequency group (features of its padding
// rows masked to zero), as in the sweeps.
template <class T, int D, int FW, int NW, bool NS, bool MASK = false>
__global__ __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(state_waves_per_eu(D, NS, NW), state_waves_per_eu(D, NS, NW))))
void k_fwd_state(FwdArgs a) {
  typedef Shape<T, D, FW, NW, NS> SH;
  typedef typename Io<T>::type IO;
  typedef RowStage<IO, D, SH::NT> StK;
  typedef RowStage<IO, SH::DV, SH::NT> StV;
  __shared__ __attribute__((aligned(16))) IO XK[StK::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) float SCK[CHUNK];   // staged: per-token scale s e(k)
  __shared__ __attribute__((aligned(16))) IO XV[StV::LDS_ELEMS];   // [token][value col]

  const WgCoord wc = wg_coord(a.pre_segs * a.sub, a.H, a.BH);   // seg: sub-segment
  const int seg = wc.seg, bh = wc.bh, h = bh % a.H;
  const int w = threadIdx.x / WAVE;
  const int fv = slice_valid<MASK, FW>(a.fvalid, w);
  const int cps = a.chunks_per_seg / a.sub;
  const int c0 = seg * cps;
  const int c1 = min(c0 + cps, a.nchunks);
  const IO* K = static_cast<const IO*>(a.K) + (size_t)bh * a.N * D;
  const IO* V = static_cast<const IO*>(a.V) + (size_t)bh * a.N * SH::DV;

  StK sk;
  StV sv;
  if (c0 < c1) {
    sk.fetch(K, c0 * CHUNK, a.N);
    sv.fetch(V, c0 * CHUNK, a.N);
  }
  const Frag<T>* wproj = FragBlock<T, D, FW, NS>::proj(a.wfrag, h, NW, w);
  const auto inv_c = inv_c_of<T>(a.tau[h]);

  f32x4 S[SH::FC][SH::DVT1];
#pragma unroll
  for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt) S[fc][dt] = zero4();
  const Frag<T> ones = ones_all<T>();
  const int g = (threadIdx.x % WAVE) / 16;

  // projection fragments: held for the whole sweep where registers allow, else
  // reloaded per chunk ahead of the staging barriers
  constexpr bool KEEP_FS = state_keeps_frags(D, NW);
  FreqSlice<T, D, FW, NS> fs;
  // held for the whole sweep: built from W by each wave (no prepared copy is needed)
  if (KEEP_FS) fs.load(a.W1 + (size_t)h * a.w_stride, NS ? a.W2 + (size_t)h * a.w_stride : nullptr, w * FW);
  for (int c = c0; c < c1; ++c) {
    const int tok0 = c * CHUNK;
    if (!KEEP_FS) fs.load_frags(wproj);
    __syncthreads();
    sk.store(XK, SCK, [&](int t, auto ssq) { return row_scale(ssq, inv_c, a.s_const, tok0 + t < a.N); });
    sv.store(XV);
    {
      const int t1 = c + 1 < c1 ? tok0 + CHUNK : tok0;   // the last chunk refetches itself (unused)
      sk.fetch(K, t1, a.N);
      sv.fetch(V, t1, a.N);
    }
    __syncthreads();
    // phi(K) with the tokens as the contraction index, straight from registers
#pragma unroll
    for (int ks = 0; ks < SH::KT; ++ks) {
      Frag<T> pk[SH::FC];
      feature_frags_rows<T, D, FW, NS, StK::LD>(fs, XK, SCK, ks, pk, fv);
      Frag<T> vf[SH::DVT];
#pragma unroll
      for (int dt = 0; dt < SH::DVT; ++dt) vf[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XV), StV::LD, 32 * ks + 4 * g, 32 * ks + 16 + 4 * g, dt * 16);
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc) {
#pragma unroll
        for (int dt = 0; dt < SH::DVT; ++dt) mma(S[fc][dt], pk[fc], vf[dt]);
        mma(S[fc][SH::DVT], pk[fc], ones);
      }
    }
  }
  float* out = a.state + ((size_t)bh * a.segments * a.sub + seg) * SH::STATE + (size_t)w * SH::WAVE_STATE;
  const int l = threadIdx.x % WAVE;
#pragma unroll
  for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
    for (int dt = 0; dt < SH::DVT1; ++dt)
      *reinterpret_cast<f32x4*>(out + ((fc * SH::DVT1 + dt) * WAVE + l) * 4) = S[fc][dt];
}

// ---------------------------------------------------------------------------
// Exclusive prefix over segments (causal) or total into segment 0 (non-causal).
// state: [BH][P][E] fp32.  Fixed summation order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_state_scan(float* state0, float* state1, int P, int sub, int E,
                                                    int causal, int reverse0, int nread0) {
  // one thread per 4 consecutive elements (E is a multiple of 256)
  const int e4 = blockIdx.x * 256 + threadIdx.x;
  if (4 * e4 >= E) return;
  const int n = P * sub;
  // blockIdx.z selects the state array: state0 in the direction reverse0,
  // state1 (backward only) in the opposite one
  const int reverse = blockIdx.z == 0 ? reverse0 : 1 - reverse0;
  float4* s = reinterpret_cast<float4*>((blockIdx.z == 0 ? state0 : state1) + (size_t)blockIdx.y * n * E) + e4;
  const size_t E4 = E / 4;
  const int nread = blockIdx.z == 0 ? nread0 : n;   // slots holding local states (scan order)
  constexpr int BATCH = 16;  // independent loads in flight per thread
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k0 = 0; k0 < n; k0 += BATCH) {
    float4 v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int k = k0 + j;
      const int p = reverse ? n - 1 - k : k;
      v[j] = k < nread ? s[(size_t)p * E4] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (causal) {
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const int k = k0 + j;
        const int p = reverse ? n - 1 - k : k;
        // first slot of each segment met in scan order: p*sub (prefix) or p*sub+sub-1 (suffix)
        if (k < n && (reverse ? (p % sub == sub - 1) : (p % sub == 0))) s[(size_t)p * E4] = acc;
        acc.x += v[j].x; acc.y += v[j].y; acc.z += v[j].z; acc.w += v[j].w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < BATCH; ++j) { acc.x += v[j].x; acc.y += v[j].y; acc.z += v[j].z; acc.w += v[j].w; }
    }
  }
  if (!causal) s[0] = acc;
}

// Total of the n local states of every slice, in the scan's order, into another
// array: src blocks of src_stride floats (n of them per slice), dst one block of
// dst_stride per slice; the first E floats of a block are summed.
__global__ __launch_bounds__(256) void k_state_sum(const float* src, int n, int src_stride, float* dst, int dst_stride,
                                                   int E) {
  const int e4 = blockIdx.x * 256 + threadIdx.x;
  if (4 * e4 >= E) return;
  const float* s = src + (size_t)blockIdx.y * n * src_stride + 4 * e4;
  f32x4 acc = zero4();
#pragma unroll 4
  for (int k = 0; k < n; ++k) acc += *reinterpret_cast<const f32x4*>(s + (size_t)k * src_stride);
  *reinterpret_cast<f32x4*>(dst + (size_t)blockIdx.y * dst_stride + 4 * e4) = acc;
}

// ---------------------------------------------------------------------------
// Sweep: carry-in state, then per chunk the readout (and, causal, the
// intra-chunk term and the state update).  Writes O and den.
//
// A chunk has two phases.  In the first the waves split the frequencies: each
// forms phi(Q) and phi(K) of its slice for the chunk's tokens, writes them and
// its bf16 copy of the state to LDS as operand fragments, and updates its
// state.  In the second they split the output: a wave takes one 16-token tile
// (and, with more waves than tiles, a part of the value columns) over all
// features.  So no partial sum crosses waves, the intra-chunk kernel matrix of
// a tile is formed once over all features (not once per slice), and the
// division and the store follow from the accumulators.
//
// Bound by vector issue and the latency of the two phases.  With the readout's
// partial sums, their reduction and the per-slice kernel matrices gone, 8
// waves of 16 frequencies at d = 64, m = 128 fit two waves per SIMD with no
// accumulator moves, and at m = 64 two workgroups share a CU.  us per sweep,
// before (4 waves of 32 frequencies, partials reduced through LDS) and after:
// d = 64, m = 128 nonstationary, B*H = 32, N = 8192: 97 and 81; stationary,
// B*H = 96, N = 1024: 44 and 39; d = 128, m = 256 (four groups, and the last
// one divides, where a pass of its own took 35): 620 and 559, and 300 as two
// groups of 128 frequencies with 8 waves.
// ---------------------------------------------------------------------------
// The work split of the second phase.
template <class T, int D, int FW, int NW, bool NS, int CH>
struct SweepShape {
  typedef Shape<T, D, FW, NW, NS, CH> SH;
  static constexpr int TT = CH / 16;                  // token tiles per chunk
  static constexpr int NFT = SH::M / 16;              // frequency tiles of all waves
  static constexpr int WPT = NW > TT ? NW / TT : 1;   // waves per token tile in the second phase
  static constexpr int NDT = (SH::DVT + WPT - 1) / WPT;   // value tiles of one of them
  static_assert(TT <= NW && NW % TT == 0, "whole token tiles per wave");
};

// ADD: add this frequency group's numerator and denominator to the sums the
// earlier groups stored; the old sums are loaded at the start of each chunk,
// so their latency overlaps the chunk's work.
// CH: tokens per chunk of the causal sweep (16, 32 or 64; the intra-chunk
// term covers j <= i within a chunk, earlier tokens enter through the carried
// state).  Token contractions run in 32-token MFMA k-steps; a 16-token chunk
// pads its k-step with zero rows (staged once, never written).
template <class T, int D, int FW, int NW, bool NS, bool CAUSAL, bool ADD, int CH, bool MASK = false>
__global__ __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(sweep_waves_per_eu(IsBf16<T>::value, D, FW * NW, NS, CAUSAL, CH))))
void k_fwd_sweep(FwdArgs a) {
  typedef SweepShape<T, D, FW, NW, NS, CH> SS;
  typedef typename SS::SH SH;
  typedef typename Io<T>::type IO;
  typedef RowStage<IO, D, SH::NT, CH> StX;
  typedef RowStage<IO, SH::DV, SH::NT, CH> StV;
  constexpr int TT = SS::TT, NFT = SS::NFT, NDT = SS::NDT;
  constexpr int KT = (CH + 31) / 32;           // 32-token k-steps per chunk
  constexpr int ROWS = KT * 32;                // token rows of the k-step operands
  static_assert(CH == 16 || CH == 32 || CH == 64, "chunk of 16, 32 or 64 tokens");
  static_assert(CAUSAL || CH == CHUNK, "the non-causal sweep uses 64-token chunks");
  constexpr int XV_N = CAUSAL ? ROWS * StV::LD : 8;
  constexpr int LDP = SH::FC * 16 + 4;     // [token][feature] rows of a wave's phi(K) block
  constexpr int PT_N = CAUSAL ? ROWS * LDP : 8;
  __shared__ __attribute__((aligned(16))) IO XQ[StX::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) IO XK[CAUSAL ? StX::LDS_ELEMS : 8];
  __shared__ __attribute__((aligned(16))) float SCQ[CH], SCK[CH];   // staged: per-token scales s e(x)
  __shared__ __attribute__((aligned(16))) IO XV[XV_N];   // [token][value col]
  __shared__ __attribute__((aligned(16))) T PT[NW][PT_N];
  __shared__ Frag<T> PQ[TT][NFT][WAVE];        // phi(Q), operand fragments
  __shared__ Frag<T> SB[SH::DVT][NFT][WAVE];   // state, operand fragments (rows = value columns)
  __shared__ Frag<T> SZ[NFT][4];               // normaliser rows of the state, all columns alike
  // Where the chunks are cut short more of a row's keys reach den through SZ than
  // through the intra-chunk matrix, and rounded once it carries more error than in
  // chunks of 64 (up to 2.5 % at N = 512).  There the cos features, whose sums are
  // large, have a low part too (two frequency tiles to an operand), in every wave, so
  // that each divides by the den that is written.  Error of den against float64,
  // nonstationary, with and without: m = 256, N = 8192 1.24e-4 and 1.78e-4, m = 128, N =
  // 1000 1.70e-4 and 2.53e-4; us per forward 450 and 450, m = 128, B*H = 96, N = 1024
  // 95.3 and 92.9 (as an operand of its own for each frequency tile, in the waves that
  // write den alone, 465 and 97).
  constexpr bool ZLOW = CAUSAL && IsBf16<T>::value && sweep_short_chunks(D, SH::M);
  __shared__ Frag<T> SZL[ZLOW ? NFT / 2 : 1][4];

  // causal: one workgroup per segment; non-causal: per group of chunks (every
  // chunk reads the same total state)
  const WgCoord wc = wg_coord(a.sweep_groups, a.H, a.BH);
  const int seg = wc.seg, bh = wc.bh, h = bh % a.H;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  const int fv = slice_valid<MASK, FW>(a.fvalid, w);
  const int nch = (a.N + CH - 1) / CH;
  const int c0 = seg * a.sweep_cps;
  const int c1 = min(c0 + a.sweep_cps, nch);
  const IO* Q = static_cast<const IO*>(a.Q) + (size_t)bh * a.N * D;
  const IO* K = static_cast<const IO*>(a.K) + (size_t)bh * a.N * D;
  const IO* V = static_cast<const IO*>(a.V) + (size_t)bh * a.N * SH::DV;
  IO* O = static_cast<IO*>(a.O) + (size_t)bh * a.N * SH::DV;
  float* den = a.den ? a.den + (size_t)bh * a.N : nullptr;
  // second phase: this wave's token tile and its part of the value columns.
  // The waves of one SIMD (w and w + 4) take tiles from both ends, so their
  // causal work adds up alike.
  const int part = w / TT;
  const int tq = part % 2 ? TT - 1 - w % TT : w % TT;

  StX sq, sk;
  StV sv;
  if (c0 < c1) {
    sq.fetch(Q, c0 * CH, a.N);
    if (CAUSAL) sk.fetch(K, c0 * CH, a.N);
    if (CAUSAL) sv.fetch(V, c0 * CH, a.N);
  }
  if (CAUSAL && CH < ROWS) {
    // zero k-step padding rows of V and of this wave's phi(K) block (both
    // zero, so no product with uninitialised LDS enters a sum)
    for (int i = threadIdx.x; i < (ROWS - CH) * StV::LD; i += SH::NT) XV[CH * StV::LD + i] = IO(0);
    for (int i = l; i < (ROWS - CH) * LDP; i += WAVE) PT[w][CH * LDP + i] = T(0.0f);
  }
  const auto inv_c = inv_c_of<T>(a.tau[h]);

  // carry-in state (exclusive prefix for causal, total for non-causal)
  f32x4 S[SH::FC][SH::DVT1];
  {
    const float* blk = a.state + (size_t)bh * a.segments * a.sub * SH::STATE + (size_t)w * SH::WAVE_STATE;
    if (a.fold) {
      // the exclusive prefix (total) of the local states, summed in the scan's order
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
        for (int dt = 0; dt < SH::DVT1; ++dt) S[fc][dt] = zero4();
      for (int k = 0; k < (CAUSAL ? seg : a.pre_segs) * a.sub; ++k) {
        const float* in = blk + (size_t)k * SH::STATE;
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
          for (int dt = 0; dt < SH::DVT1; ++dt)
            S[fc][dt] += *reinterpret_cast<const f32x4*>(in + ((fc * SH::DVT1 + dt) * WAVE + l) * 4);
      }
    } else {
      const float* in = blk + (size_t)(CAUSAL ? seg * a.sub : 0) * SH::STATE;
#pragma unroll
      for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
        for (int dt = 0; dt < SH::DVT1; ++dt)
          S[fc][dt] = *reinterpret_cast<const f32x4*>(in + ((fc * SH::DVT1 + dt) * WAVE + l) * 4);
    }
  }
  const Frag<T> ones = ones_all<T>();
  // projection fragments, held for the whole sweep: built from W by each wave
  FreqSlice<T, D, FW, NS> fs;
  fs.load(a.W1 + (size_t)h * a.w_stride, NS ? a.W2 + (size_t)h * a.w_stride : nullptr, w * FW);
  // this wave's rows of the state as operand fragments, for every wave
  auto store_state = [&]() {
#pragma unroll
    for (int ft = 0; ft < SH::FT; ++ft) {
#pragma unroll
      for (int dt = 0; dt < SH::DVT; ++dt)
        SB[dt][w * SH::FT + ft][l] = pair_tiles<T>(S[2 * ft][dt], S[2 * ft + 1][dt]);
      const Frag<T> z = pair_tiles<T>(S[2 * ft][SH::DVT], S[2 * ft + 1][SH::DVT]);
      if (r == 0) SZ[w * SH::FT + ft][g] = z;
      if constexpr (ZLOW) {
        static_assert(SH::FT == 1 && NFT % 2 == 0, "two waves to a low operand");
        T* o = reinterpret_cast<T*>(&SZL[w / 2][g]) + 4 * (w % 2);
        if (r == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = (T)(S[0][SH::DVT][i] - z.get(i));
        }
      }
    }
  };
  if (!CAUSAL) store_state();   // ordered by the first staging barrier

  for (int c = c0; c < c1; ++c) {
    const int tok0 = c * CH;
    // no barrier before the staging stores: every read of the staging buffers
    // is in the first phase, which the previous chunk's second barrier ends
    sq.store(XQ, SCQ, [&](int t, auto ssq) { return row_scale(ssq, inv_c, a.s_const, tok0 + t < a.N); });
    if (CAUSAL) {
      sk.store(XK, SCK, [&](int t, auto ssq) { return row_scale(ssq, inv_c, a.s_const, tok0 + t < a.N); });
      sv.store(XV);
    }
    __syncthreads();   // rows staged; the previous chunk's fragments are read
    // next chunk's rows
    {
      const int t1 = c + 1 < c1 ? tok0 + CH : tok0;   // the last chunk refetches itself (unused)
      sq.fetch(Q, t1, a.N);
      if (CAUSAL) sk.fetch(K, t1, a.N);
      if (CAUSAL) sv.fetch(V, t1, a.N);
    }
    // the earlier groups' sums for this wave's rows (rows past N read zero)
    const RowBuf nb(a.acc_num + (size_t)bh * a.N * SH::DV, SH::DV, ADD ? tok0 : 0, a.N, CH);
    const RowBuf db(a.acc_den + (size_t)bh * a.N, 1, ADD ? tok0 : 0, a.N, CH);
    f32x4 old_n[ADD ? NDT : 1];
    float old_d = 0.f;
    if (ADD) {
#pragma unroll
      for (int k = 0; k < NDT; ++k)
        if (part * NDT + k < SH::DVT)
          old_n[k] = nb.load_f4(((tq * 16 + r) * SH::DV + (part * NDT + k) * 16 + 4 * g) * 4);
      old_d = db.load_f1((tq * 16 + r) * 4);
    }

    if (CAUSAL) store_state();   // the state before this chunk
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      ProjT<T> p[SH::PR];
      float sc;
      project_tile_lds<T, D, FW, NS, StX::LD>(fs, XQ, SCQ, tt, p, sc);
#pragma unroll
      for (int ft = 0; ft < SH::FT; ++ft) PQ[tt][w * SH::FT + ft][l] = features<T, SH::FT, NS>(p, ft, sc, fv);
    }
    Frag<T> vf[CAUSAL ? NDT : 1][KT];
    if (CAUSAL) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        ProjT<T> p[SH::PR];
        float sc;
        project_tile_lds<T, D, FW, NS, StX::LD>(fs, XK, SCK, tt, p, sc);
#pragma unroll
        for (int ft = 0; ft < SH::FT; ++ft)
          store_frag_nm<T>(PT[w], LDP, tt * 16, (2 * ft) * 16, (2 * ft + 1) * 16, features<T, SH::FT, NS>(p, ft, sc, fv));
      }
      // state update S' += phi(K)^T [V | 1] with this wave's transposed phi(K)
#pragma unroll
      for (int ks = 0; ks < KT; ++ks) {
        Frag<T> va[SH::DVT];
#pragma unroll
        for (int dt = 0; dt < SH::DVT; ++dt)
          va[dt] = lds_tr_frag<T>(reinterpret_cast<const T*>(XV), StV::LD, 32 * ks + 4 * g, 32 * ks + 16 + 4 * g, dt * 16);
#pragma unroll
        for (int fc = 0; fc < SH::FC; ++fc) {
          const Frag<T> pkt = lds_tr_frag<T>(PT[w], LDP, 32 * ks + 4 * g, 32 * ks + 16 + 4 * g, fc * 16);
#pragma unroll
          for (int dt = 0; dt < SH::DVT; ++dt) mma_rows<CH>(S[fc][dt], pkt, va[dt]);
          mma_rows<CH>(S[fc][SH::DVT], pkt, ones);
        }
      }
      // this wave's value columns for the second phase
#pragma unroll
      for (int k = 0; k < NDT; ++k)
#pragma unroll
        for (int ks = 0; ks < KT; ++ks) {
          const int dt = part * NDT + k < SH::DVT ? part * NDT + k : 0;
          vf[k][ks] = lds_tr_frag<T>(reinterpret_cast<const T*>(XV), StV::LD, 32 * ks + 4 * g, 32 * ks + 16 + 4 * g, dt * 16);
        }
    }
    __syncthreads();   // every wave's fragments complete

    if (part * NDT < SH::DVT) {
      Frag<T> pq[NFT];
#pragma unroll
      for (int ft = 0; ft < NFT; ++ft) pq[ft] = PQ[tq][ft][l];
      // intra-chunk kernel matrix, transposed: rows = key tokens, cols = query tokens
      // (as a high and a low operand: rounded once, a whole row of it would
      // carry more error than the features it is made of)
      Frag<T> ap[CAUSAL ? KT : 1], al[CAUSAL ? KT : 1];
      if (CAUSAL) {
        f32x4 at[2 * KT];
#pragma unroll
        for (int tk = 0; tk < 2 * KT; ++tk) {
          at[tk] = zero4();
          if (tk < TT && tk <= tq) {
#pragma unroll
            for (int ft = 0; ft < NFT; ++ft)
              mma(at[tk],
                  load_frag_nm<T>(PT[ft / SH::FT], LDP, tk * 16, (2 * (ft % SH::FT)) * 16, (2 * (ft % SH::FT) + 1) * 16),
                  pq[ft]);
            if (tk == tq) {
#pragma unroll
              for (int i = 0; i < 4; ++i) at[tk][i] = 4 * g + i > r ? 0.f : at[tk][i];
            }
          }
        }
#pragma unroll
        for (int ks = 0; ks < KT; ++ks) split_pair<T>(at[2 * ks], at[2 * ks + 1], ap[ks], al[ks]);
      }
      // (fp32: the odd frequency tiles in sums of their own, shorter to round)
      constexpr int NSUM = IsBf16<T>::value ? 1 : 2;
      f32x4 accs[NSUM][NDT], zn = zero4();
#pragma unroll
      for (int p = 0; p < NSUM; ++p)
#pragma unroll
        for (int k = 0; k < NDT; ++k) accs[p][k] = zero4();
      f32x4 (&acc)[NDT] = accs[0];
      f32x4 zl = zero4();   // den's share of the low operands
      auto intra = [&]() {
#pragma unroll
        for (int ks = 0; ks < KT; ++ks)
          if (32 * ks <= 16 * tq + 15) {
#pragma unroll
            for (int k = 0; k < NDT; ++k) {
              mma_tree<CH>(acc[k], vf[k][ks], ap[ks]);
              if (IsBf16<T>::value) mma(acc[k], vf[k][ks], al[ks]);
            }
            if (IsBf16<T>::value) {
              mma(zn, ones, ap[ks]);
              mma(zl, ones, al[ks]);
            }
          }
      };
      // fp32: the intra-chunk share first, while the sums are small (den's error
      // against float64 1.56e-7 after the state's share, 1.51e-7 before it).  In
      // bf16 the state's products fill the wait for the kernel matrix: the
      // intra-chunk share first costs 1 %, and 5 % in chunks of 16 tokens.
      if (CAUSAL && !IsBf16<T>::value) intra();
#pragma unroll
      for (int ft = 0; ft < NFT; ++ft) {
#pragma unroll
        for (int k = 0; k < NDT; ++k)
          if (SH::DVT % NDT == 0 || part * NDT + k < SH::DVT) mma(accs[ft % NSUM][k], SB[part * NDT + k][ft][l], pq[ft]);
        if (IsBf16<T>::value) mma(zn, SZ[ft][g], pq[ft]);
      }
      if constexpr (NSUM == 2) {
#pragma unroll
        for (int k = 0; k < NDT; ++k) acc[k] += accs[1][k];
      }
      if constexpr (ZLOW) {
#pragma unroll
        for (int p = 0; p < NFT / 2; ++p) {
          Frag<T> c2;   // cos features of two frequency tiles
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            c2.v[i] = pq[2 * p].v[i];
            c2.v[4 + i] = pq[2 * p + 1].v[i];
          }
          mma(zl, SZL[p][g], c2);
        }
      }
      if (CAUSAL && IsBf16<T>::value) intra();
      // acc[k]: rows = value columns, column = token r; every row of the
      // normaliser tile holds den of token r
      float dn = zn[0];
      if (CAUSAL && IsBf16<T>::value) dn += finite_low(zl[0]);
      if constexpr (!IsBf16<T>::value) {
        // fp32: on the vector units, in float64.  As matrix products the waves of a token
        // tile would each form 16 equal rows of it, 40 of a wave's 112 in chunks of 16.
        // (In fp32 chains den lost accuracy where it cancels.)  us per forward, B*H = 32,
        // N = 1023 nonstationary, before and after: chunks of 16, with the padding out of
        // the k-steps, 69.3 and 63.5, of 32 56.5 and 55.5; error of den against float64
        // 1.55e-7 and 1.38e-7.
        double t[2] = {0.0, 0.0};
        if (CAUSAL) {
#pragma unroll
          for (int ks = 0; ks < KT; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) t[j % 2] += (double)ap[ks].get(j);
        }
#pragma unroll
        for (int ft = 0; ft < NFT; ++ft) {
          const Frag<T> z = SZ[ft][g];
#pragma unroll
          for (int j = 0; j < 8; ++j) t[j % 2] = fma((double)pq[ft].get(j), (double)z.get(j), t[j % 2]);
        }
        double s = t[0] + t[1];
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        dn = (float)s;
      }
      if (ADD) dn += old_d;
      if (ADD ? a.acc == 2 : a.acc != 0) {
        // one frequency group's share of the numerator and denominator
#pragma unroll
        for (int k = 0; k < NDT; ++k)
          if (SH::DVT % NDT == 0 || part * NDT + k < SH::DVT) {
            if (ADD) acc[k] += old_n[k];
            RowBuf(a.acc_num + (size_t)bh * a.N * SH::DV, SH::DV, tok0, a.N, CH)
                .store_f4(((tq * 16 + r) * SH::DV + (part * NDT + k) * 16 + 4 * g) * 4, acc[k]);
          }
        if (part == 0 && g == 0) RowBuf(a.acc_den + (size_t)bh * a.N, 1, tok0, a.N, CH).store_f1((tq * 16 + r) * 4, dn);
      } else {
        // one reciprocal per row (v_rcp_f32, 1 ulp); den = 0 gives inf/NaN as num/0 does
        const float inv = __builtin_amdgcn_rcpf(dn);
        const RowBuf ob(O, SH::DV, tok0, a.N, CH);
#pragma unroll
        for (int k = 0; k < NDT; ++k)
          if (SH::DVT % NDT == 0 || part * NDT + k < SH::DVT) {
            if (ADD) acc[k] += old_n[k];
            ob.store_io4(O, ((tq * 16 + r) * SH::DV + (part * NDT + k) * 16 + 4 * g) * (int)sizeof(IO), acc[k] * inv);
          }
        if (den && part == 0 && g == 0) RowBuf(den, 1, tok0, a.N, CH).store_f1((tq * 16 + r) * 4, dn);
      }
    }
  }
  if (CAUSAL && a.state_out && seg == a.sweep_groups - 1) {
    // causal prefill: the last segment ends with the state of the whole
    // sequence (an empty trailing segment holds it as its carry-in).  Tile
    // (fc, dt) has rows = features 4g+i of feature tile fc (fc = 2ft: cos of
    // frequency tile ft, 2ft+1: its sin) and cols = value columns; the
    // normaliser tile holds z in every column.
    const size_t F2 = 2 * (size_t)a.state_m;
    const int sdv = a.state_dv;   // value columns of the state layout, <= SH::DV
    float* so = a.state_out + (size_t)bh * F2 * (sdv + 1);
    float* zo = so + F2 * sdv;
#pragma unroll
    for (int fc = 0; fc < SH::FC; ++fc)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int fl = w * FW + (fc / 2) * 16 + 4 * g + i;   // row within the group
        if (fl >= a.fvalid) continue;   // a padding row of a padded group
        const int f = a.state_f0 + fl;
        const size_t row = (fc % 2) ? (size_t)a.state_m + f : (size_t)f;
#pragma unroll
        for (int dt = 0; dt < SH::DVT; ++dt)
          if (dt * 16 + r < sdv) so[row * sdv + dt * 16 + r] = S[fc][dt][i];
        if (r == 0) zo[row] = S[fc][SH::DVT][i];
      }
  }
}

// Four consecutive values of one row as one vector store in the io dtype.
template <class IO>
__device__ __forceinline__ void store4(IO* p, const float (&v)[4]);
template <>
__device__ __forceinline__ void store4<u16>(u16* p, const float (&v)[4]) {
  const uint2 w = make_uint2((uint32_t)float_to_bf16_bits(v[0]) | ((uint32_t)float_to_bf16_bits(v[1]) << 16),
                             (uint32_t)float_to_bf16_bits(v[2]) | ((uint32_t)float_to_bf16_bits(v[3]) << 16));
  *reinterpret_cast<uint2*>(p) = w;
}
template <>
__device__ __forceinline__ void store4<float>(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// ---------------------------------------------------------------------------
// Non-causal readout with the tokens split across waves (bf16, m_eff <= 64).
// Every chunk reads the same total state, so each of the four waves takes one
// 16-token tile of a 64-token chunk over all 2m features: the total state is
// held by every wave as bf16 operand fragments (rows = value columns, k = the
// 32 features of one frequency tile, [cos | sin] as the feature fragments),
// and each wave projects its tokens onto all m frequencies.  No partial sums
// cross waves, so the only barrier per chunk is the staging one.
// ---------------------------------------------------------------------------
template <class T, int D, int M, bool NS, bool MASK = false>
__global__ __launch_bounds__(4 * WAVE) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_fwd_readout(FwdArgs a) {
  constexpr int NWR = 4;                        // waves: one 16-token tile each
  constexpr int FT = M / 16;                    // frequency tiles (all of them)
  constexpr int DVT = D / 16, DVT1 = DVT + 1;
  typedef FreqSlice<T, D, M, NS> FS;
  typedef Shape<T, D, 16, M / 16, NS> SS;       // the state pre-pass's split: 16 frequencies per wave
  typedef typename Io<T>::type IO;
  typedef RowStage<IO, D, NWR * WAVE> StX;
  static_assert(CHUNK == 16 * NWR, "one token tile per wave");
  __shared__ __attribute__((aligned(16))) IO XQ2[2][StX::LDS_ELEMS];
  __shared__ typename StX::Ssq SSQ2[2][CHUNK];

  const WgCoord wc = wg_coord(a.sweep_groups, a.H, a.BH);
  const int seg = wc.seg, bh = wc.bh, h = bh % a.H;
  const int w = threadIdx.x / WAVE, l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  const int c0 = seg * a.sweep_cps;
  const int c1 = min(c0 + a.sweep_cps, a.nchunks);
  const IO* Q = static_cast<const IO*>(a.Q) + (size_t)bh * a.N * D;
  IO* O = static_cast<IO*>(a.O) + (size_t)bh * a.N * D;
  float* den = a.den ? a.den + (size_t)bh * a.N : nullptr;

  StX sq;
  if (c0 < c1) sq.fetch(Q, c0 * CHUNK, a.N);
  const auto inv_c = inv_c_of<T>(a.tau[h]);
  // total state (slot 0 of this slice): pre-pass wave ft holds
  // frequency tile ft, its tile fc = 0 the cos features and fc = 1 the sin ones
  Frag<T> sf[DVT1][FT];
  {
    const float* in = a.state + (size_t)bh * a.segments * a.sub * SS::STATE;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int dt = 0; dt < DVT1; ++dt) {
        const float* blk = in + (size_t)ft * SS::WAVE_STATE;
        const f32x4 cs = *reinterpret_cast<const f32x4*>(blk + ((0 * DVT1 + dt) * WAVE + l) * 4);
        const f32x4 sn = *reinterpret_cast<const f32x4*>(blk + ((1 * DVT1 + dt) * WAVE + l) * 4);
        sf[dt][ft] = pair_tiles<T>(cs, sn);
      }
  }
  FS fs;
  fs.load(a.W1 + (size_t)h * a.w_stride, NS ? a.W2 + (size_t)h * a.w_stride : nullptr, 0);

  for (int c = c0; c < c1; ++c) {
    // double-buffered staging: the chunk that last read this buffer (two back)
    // is separated from this store by the previous chunk's barrier
    const int par = (c - c0) & 1;
    IO* XQ = XQ2[par];
    typename StX::Ssq* SSQ = SSQ2[par];
    const int tok0 = c * CHUNK;
    sq.store(XQ, SSQ);
    sq.fetch(Q, c + 1 < c1 ? tok0 + CHUNK : tok0, a.N);   // the last chunk refetches itself (unused)
    __syncthreads();
    ProjT<T> p[FS::PR];
    typename StX::Ssq ssq;
    project_tile_lds<T, D, M, NS, StX::LD>(fs, XQ, SSQ, w, p, ssq);
    const int tok = tok0 + w * 16 + r;
    const float sc = row_scale(ssq, inv_c, a.s_const, tok < a.N);
    f32x4 acc[DVT1];
#pragma unroll
    for (int dt = 0; dt < DVT1; ++dt) acc[dt] = zero4();
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const Frag<T> pq = features<T, FT, NS>(p, ft, sc, MASK ? a.fvalid : M);
#pragma unroll
      for (int dt = 0; dt < DVT1; ++dt) mma(acc[dt], sf[dt][ft], pq);
    }
    // acc[dt]: rows = value columns dt*16 + 4g + i, column = token r; every
    // row of the normaliser tile holds den
    const float dn = acc[DVT][0];
    const float inv = __builtin_amdgcn_rcpf(dn);   // den = 0 gives inf/NaN as num/0 does
    const RowBuf ob(O, D, tok0, a.N, CHUNK);
#pragma unroll
    for (int dt = 0; dt < DVT; ++dt)
      ob.store_io4(O, ((w * 16 + r) * D + dt * 16 + 4 * g) * (int)sizeof(IO), acc[dt] * inv);
    if (den && g == 0) RowBuf(den, 1, tok0, a.N, CHUNK).store_f1((w * 16 + r) * 4, dn);
  }
}

// ---------------------------------------------------------------------------
// Standalone feature map: Phi [B,H,N,2m], [cos | sin] blocks.  A workgroup
// walks a.chunks_per_seg consecutive chunks of one (b,h) slice with its
// frequency fragments built once; each lane writes its four consecutive
// features of a block as one vector store.
// ---------------------------------------------------------------------------
// The chunk's X rows are staged through LDS (prefetched a chunk ahead), every
// wave projects them for its frequency slice, and the features are gathered
// as [token][feature] rows in LDS, then written out as whole 16-byte vectors.
// FULL: the launch fills all M frequencies (every m but a last slice's), so a
// vector's place is known at compile time: the divisions by a row's vectors
// were half of the kernel's instructions (us per call of B*H = 96, N = 1000, d =
// 64, m = 128: 26 before, 20.6 after).
template <class T, int D, int FW, int NW, bool NS, bool FULL>
__global__ __launch_bounds__(NW * WAVE) void k_feature_map(FwdArgs a) {
  typedef Shape<T, D, FW, NW, NS> SH;
  typedef typename Io<T>::type IO;
  typedef RowStage<IO, D, SH::NT> StX;
  constexpr int F = 2 * SH::M;                 // features per staged row
  constexpr int VEC = 16 / (int)sizeof(IO);    // elements per 16-byte vector
  constexpr int LDF = F + VEC;                 // row stride of the staged features
  __shared__ __attribute__((aligned(16))) IO XL[StX::LDS_ELEMS];
  __shared__ typename StX::Ssq SSQ[CHUNK];
  __shared__ __attribute__((aligned(16))) IO PH[CHUNK * LDF];
  const int bh = blockIdx.y, h = bh % a.H;
  const int w = threadIdx.x / WAVE, l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  // this launch covers frequencies [state_f0, state_f0 + fvalid) of state_m
  // (fvalid <= M, a multiple of 16): their cos and sin columns of rows of
  // 2 state_m features
  const int fv = FULL ? SH::M : a.fvalid, mo = a.state_m, f0o = a.state_f0;
  const int vrow = 2 * fv / VEC;               // output vectors per row
  const int nvo = CHUNK * vrow;
  constexpr int NVO = (CHUNK * F / VEC + SH::NT - 1) / SH::NT;   // vectors per thread (at most)
  const IO* X = static_cast<const IO*>(blockIdx.z ? a.K : a.Q) + (size_t)bh * a.N * D;
  IO* Phi = static_cast<IO*>(blockIdx.z ? a.O2 : a.O) + (size_t)bh * a.N * 2 * mo;
  const int c0 = blockIdx.x * a.chunks_per_seg;
  const int c1 = min(c0 + a.chunks_per_seg, a.nchunks);
  StX sx;
  if (c0 < c1) sx.fetch(X, c0 * CHUNK, a.N);
  FreqSlice<T, D, FW, NS> fs;   // frequencies past fvalid load as zero rows (their columns are not written)
  fs.template load<true>(a.W1 + (size_t)h * a.w_stride, NS ? a.W2 + (size_t)h * a.w_stride : nullptr, w * FW, fv);
  const auto inv_c = inv_c_of<T>(a.tau[h]);
  for (int c = c0; c < c1; ++c) {
    const int tok0 = c * CHUNK;
    // no barrier: the previous chunk's reads of XL ended before its last barrier
    sx.store(XL, SSQ);
    sx.fetch(X, c + 1 < c1 ? tok0 + CHUNK : tok0, a.N);   // the last chunk refetches itself (unused)
    __syncthreads();   // rows staged; the previous chunk's features are read
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      ProjT<T> p[SH::PR];
      typename StX::Ssq ssq;
      project_tile_lds<T, D, FW, NS, StX::LD>(fs, XL, SSQ, tt, p, ssq);
      // the values are produced in fp32 and rounded once to the io dtype
      const float sc = row_scale(ssq, inv_c, a.s_const, tok0 + tt * 16 + r < a.N);
      IO* row = PH + (tt * 16 + r) * LDF;
#pragma unroll
      for (int ft = 0; ft < SH::FT; ++ft) {
        const Frag<float> f = features<float, SH::FT, NS>(p, ft, sc);
        const int f0 = w * FW + ft * 16 + 4 * g;
        const float cv[4] = {f.get(0), f.get(1), f.get(2), f.get(3)};
        const float sv[4] = {f.get(4), f.get(5), f.get(6), f.get(7)};
        store4<IO>(row + f0, cv);
        store4<IO>(row + SH::M + f0, sv);
      }
    }
    __syncthreads();
    const RowBuf ob(Phi, 2 * mo, tok0, a.N, CHUNK);   // drops the rows past N
#pragma unroll
    for (int k = 0; k < NVO; ++k) {
      const int v = threadIdx.x + k * SH::NT;
      if ((!FULL || CHUNK * F / VEC % SH::NT != 0) && v >= nvo) break;
      const int t = v / vrow, j = v % vrow;
      const int part = j / (fv / VEC), cv = j % (fv / VEC);   // cos block, then sin block
      ob.store16((t * 2 * mo + part * mo + f0o + cv * VEC) * (int)sizeof(IO),
                 *reinterpret_cast<const uint4*>(PH + t * LDF + part * SH::M + cv * VEC));
    }
  }
}

// ---------------------------------------------------------------------------
// Frequency rows of a padded group: dst[h][rows][d] holds the group's
// rows_valid rows of W, then zero rows (their features are masked to zero).
// One thread per 4 elements.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pad_rows(const float* src, float* dst, int rows_valid, int rows, int d,
                                                  int src_stride) {
  const int h = blockIdx.y;
  const int i4 = blockIdx.x * 256 + threadIdx.x;
  if (4 * i4 >= rows * d) return;
  const int row = 4 * i4 / d;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (row < rows_valid) v = *reinterpret_cast<const float4*>(src + (size_t)h * src_stride + 4 * i4);
  *reinterpret_cast<float4*>(dst + ((size_t)h * rows) * d + 4 * i4) = v;
}

hipError_t launch_pad_rows(const float* src, float* dst, int H, int rows_valid, int rows, int d, int src_stride,
                           hipStream_t st) {
  if (d % 4 != 0) return hipErrorInvalidValue;
  k_pad_rows<<<dim3((rows * d / 4 + 255) / 256, H), 256, 0, st>>>(src, dst, rows_valid, rows, d, src_stride);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Column padding and cropping between row-major matrices of two widths, in
// 16-byte units: dst[r][u] = src[r][u] for u < us, zero for us <= u < ud.
// One thread per 16-byte unit of dst.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy_cols(const uint4* src, int us, uint4* dst, int ud, size_t rows) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows * (size_t)ud) return;
  const size_t r = i / (size_t)ud;
  const int u = (int)(i - r * (size_t)ud);
  dst[i] = u < us ? src[r * (size_t)us + u] : make_uint4(0u, 0u, 0u, 0u);
}

hipError_t launch_copy_cols(const void* src, int cols_src, void* dst, int cols_dst, size_t rows, int elem_bytes,
                            hipStream_t st) {
  if (elem_bytes <= 0 || (cols_src * elem_bytes) % 16 != 0 || (cols_dst * elem_bytes) % 16 != 0)
    return hipErrorInvalidValue;
  const int us = cols_src * elem_bytes / 16, ud = cols_dst * elem_bytes / 16;
  const size_t n = rows * (size_t)ud;
  if (n == 0) return hipSuccess;
  const size_t blocks = (n + 255) / 256;
  if (blocks > 0x7fffffffULL) return hipErrorInvalidValue;
  // a crop reads us units of each source row and copies only the first ud of them
  k_copy_cols<<<dim3((unsigned)blocks), 256, 0, st>>>(static_cast<const uint4*>(src), us,
                                                      static_cast<uint4*>(dst), ud, rows);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Host-side dispatch.
// ---------------------------------------------------------------------------
// The token-split readout serves bf16 shapes whose projection onto all m
// frequencies fits one wave's registers (m_eff <= 64, state split 4 x 16).
template <class T, int D, int FW, int NW, bool NS>
struct ReadoutSplit {
  static constexpr bool value = IsBf16<T>::value && !NS && FW * NW == 64 && FW == 16 && D <= 64;
};

template <class T, int D, int FW, int NW, bool NS, bool ADD, bool MASK>
static void launch_sweep(const FwdArgs& a, bool causal, dim3 grid, hipStream_t st) {
  typedef Shape<T, D, FW, NW, NS> SH;
  if constexpr (!ADD && ReadoutSplit<T, D, FW, NW, NS>::value) {
    if (!causal && a.acc == 0) {   // it writes O itself, not a group's sums
      k_fwd_readout<T, D, FW * NW, NS, MASK><<<grid, 4 * WAVE, 0, st>>>(a);
      return;
    }
  }
  if (!causal) {
    k_fwd_sweep<T, D, FW, NW, NS, false, ADD, CHUNK, MASK><<<grid, SH::NT, 0, st>>>(a);
  } else if (a.sweep_chunk == 16) {
    k_fwd_sweep<T, D, FW, NW, NS, true, ADD, 16, MASK><<<grid, SH::NT, 0, st>>>(a);
  } else if (a.sweep_chunk == 32) {
    k_fwd_sweep<T, D, FW, NW, NS, true, ADD, 32, MASK><<<grid, SH::NT, 0, st>>>(a);
  } else if constexpr (!sweep_short_chunks(D, FW * NW)) {
    k_fwd_sweep<T, D, FW, NW, NS, true, ADD, 64, MASK><<<grid, SH::NT, 0, st>>>(a);
  }
}

template <class T, int D, int FW, int NW, bool NS>
static hipError_t run_fwd_t(const FwdArgs& a, bool causal, hipStream_t st) {
  typedef Shape<T, D, FW, NW, NS> SH;
  const dim3 grid(a.sweep_groups * a.BH);
  const dim3 pgrid(a.pre_segs * a.sub * a.BH);
  // prepared fragments serve the state pre-pass where it reloads them per
  // chunk; the other forward kernels build theirs from W once
  if (!state_keeps_frags(D, NW)) k_prep_freqs<T, D, FW, NW, NS><<<dim3(a.H, NW, 1), WAVE, 0, st>>>(a.W1, a.W2, a.wfrag, a.w_stride);
  timing_mark(KC_FWD_STATE, st, true);
  // a padded frequency group (it runs first, so it never adds) takes the
  // masking kernel variants
  const bool masked = a.fvalid < FW * NW;
  constexpr bool CAN_MASK = group_can_pad(D, FW * NW);
  if (masked && (!CAN_MASK || a.acc >= 2)) return hipErrorInvalidValue;
  if (causal && sweep_short_chunks(D, FW * NW) && a.sweep_chunk > 32) return hipErrorInvalidValue;
  if (pgrid.x > 0) {
    if constexpr (CAN_MASK) {
      if (masked) k_fwd_state<T, D, FW, NW, NS, true><<<pgrid, SH::NT, 0, st>>>(a);
      else k_fwd_state<T, D, FW, NW, NS, false><<<pgrid, SH::NT, 0, st>>>(a);
    } else {
      k_fwd_state<T, D, FW, NW, NS, false><<<pgrid, SH::NT, 0, st>>>(a);
    }
  }
  timing_mark(KC_FWD_STATE, st, false);
  if (!a.fold) {
    const hipError_t e =
        launch_state_scan(a.state, nullptr, a.BH, a.segments, a.sub, SH::STATE, causal, st, a.pre_segs * a.sub);
    if (e != hipSuccess) return e;
  }
  timing_mark(KC_FWD_SWEEP, st, true);
  // a later frequency group adds to the earlier groups' sums
  if (a.acc >= 2) {
    launch_sweep<T, D, FW, NW, NS, true, false>(a, causal, grid, st);
  } else if (masked) {
    if constexpr (CAN_MASK) launch_sweep<T, D, FW, NW, NS, false, true>(a, causal, grid, st);
  } else {
    launch_sweep<T, D, FW, NW, NS, false, false>(a, causal, grid, st);
  }
  timing_mark(KC_FWD_SWEEP, st, false);
  return hipGetLastError();
}

template <class T, int D, int FW, int NW, bool NS>
static hipError_t run_fmap_t(const FwdArgs& a, hipStream_t st) {
  typedef Shape<T, D, FW, NW, NS> SH;
  dim3 grid((a.nchunks + a.chunks_per_seg - 1) / a.chunks_per_seg, a.BH, a.K ? 2 : 1);
  timing_mark(KC_FEATURE_MAP, st, true);
  if (a.fvalid == SH::M) k_feature_map<T, D, FW, NW, NS, true><<<grid, SH::NT, 0, st>>>(a);
  else k_feature_map<T, D, FW, NW, NS, false><<<grid, SH::NT, 0, st>>>(a);
  timing_mark(KC_FEATURE_MAP, st, false);
  return hipGetLastError();
}

template <class T, int D, int FW, int NW>
static hipError_t run_attn_v(const FwdArgs& a, bool ns, bool causal, hipStream_t st) {
  return ns ? run_fwd_t<T, D, FW, NW, true>(a, causal, st) : run_fwd_t<T, D, FW, NW, false>(a, causal, st);
}
template <class T, int D, int FW, int NW>
static hipError_t run_fmap_v(const FwdArgs& a, bool ns, hipStream_t st) {
  return ns ? run_fmap_t<T, D, FW, NW, true>(a, st) : run_fmap_t<T, D, FW, NW, false>(a, st);
}

// Feature map shapes (d, m) and attention shapes (d, m of one frequency group).
hipError_t launch_fwd(const FwdArgs& a, const KernelShape& ks, bool fmap, hipStream_t st) {
  const bool ns = ks.nonstationary, causal = ks.causal;
  if (fmap) {
    if (ks.bf16) {
      if (ks.d == 32 && ks.m == 64) return run_fmap_v<__bf16, 32, 16, 4>(a, ns, st);
      if (ks.d == 64 && ks.m == 64) return run_fmap_v<__bf16, 64, 16, 4>(a, ns, st);
      if (ks.d == 64 && ks.m == 128) return run_fmap_v<__bf16, 64, 16, 8>(a, ns, st);
      if (ks.d == 128 && ks.m == 256) return run_fmap_v<__bf16, 128, 32, 8>(a, ns, st);
    } else {
      if (ks.d == 32 && ks.m == 64) return run_fmap_v<float, 32, 16, 4>(a, ns, st);
    }
    return hipErrorInvalidValue;
  }
  if (ks.bf16) {
    if (ks.d == 32 && ks.m == 64) return run_attn_v<__bf16, 32, 16, 4>(a, ns, causal, st);
    if (ks.d == 32 && ks.m == 128) return run_attn_v<__bf16, 32, 16, 8>(a, ns, causal, st);
    if (ks.d == 64 && ks.m == 64) return run_attn_v<__bf16, 64, 16, 4>(a, ns, causal, st);
    if (ks.d == 64 && ks.m == 128) return run_attn_v<__bf16, 64, 16, 8>(a, ns, causal, st);
    if (ks.d == 128 && ks.m == 64) return run_attn_v<__bf16, 128, 16, 4>(a, ns, causal, st);
    if (ks.d == 128 && ks.m == 128) return run_attn_v<__bf16, 128, 16, 8>(a, ns, causal, st);
  } else {
    if (ks.d == 32 && ks.m == 64) return run_attn_v<float, 32, 16, 4>(a, ns, causal, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_state_scan(float* state, float* state_rev, int BH, int P, int sub, int E, bool causal,
                             hipStream_t st, int nread) {
  if (E % 4 != 0) return hipErrorInvalidValue;   // the scan moves 4 floats per thread
  dim3 sgrid((E / 4 + 255) / 256, BH, (state && state_rev) ? 2 : 1);
  timing_mark(KC_SCAN, st, true);
  if (state)
    k_state_scan<<<sgrid, 256, 0, st>>>(state, state_rev, P, sub, E, causal ? 1 : 0, 0, nread);
  else
    k_state_scan<<<sgrid, 256, 0, st>>>(state_rev, nullptr, P, sub, E, causal ? 1 : 0, 1, P * sub);
  timing_mark(KC_SCAN, st, false);
  return hipGetLastError();
}

hipError_t launch_state_sum(const float* src, int n, int src_stride, float* dst, int dst_stride, int BH, int E,
                            hipStream_t st) {
  if (E % 4 != 0 || src_stride % 4 != 0 || dst_stride % 4 != 0) return hipErrorInvalidValue;
  timing_mark(KC_SCAN, st, true);
  k_state_sum<<<dim3((E / 4 + 255) / 256, BH), 256, 0, st>>>(src, n, src_stride, dst, dst_stride, E);
  timing_mark(KC_SCAN, st, false);
  return hipGetLastError();
}

template <class T, int D, int FW, bool NS>
static size_t wfrag_bytes_t(int H, int NW) {
  return (size_t)H * NW * FragBlock<T, D, FW, NS>::PER_WAVE * sizeof(Frag<T>);
}

size_t wfrag_bytes(const KernelShape& ks, int H) {
  const bool ns = ks.nonstationary;
  if (ks.bf16) {
    if (ks.d == 32 && ks.m == 64) return ns ? wfrag_bytes_t<__bf16, 32, 16, true>(H, 4) : wfrag_bytes_t<__bf16, 32, 16, false>(H, 4);
    if (ks.d == 32 && ks.m == 128) return ns ? wfrag_bytes_t<__bf16, 32, 16, true>(H, 8) : wfrag_bytes_t<__bf16, 32, 16, false>(H, 8);
    if (ks.d == 64 && ks.m == 64) return ns ? wfrag_bytes_t<__bf16, 64, 16, true>(H, 4) : wfrag_bytes_t<__bf16, 64, 16, false>(H, 4);
    if (ks.d == 64 && ks.m == 128) return ns ? wfrag_bytes_t<__bf16, 64, 16, true>(H, 8) : wfrag_bytes_t<__bf16, 64, 16, false>(H, 8);
    if (ks.d == 128 && ks.m == 64) return ns ? wfrag_bytes_t<__bf16, 128, 16, true>(H, 4) : wfrag_bytes_t<__bf16, 128, 16, false>(H, 4);
  } else {
    if (ks.d == 32 && ks.m == 64) return ns ? wfrag_bytes_t<float, 32, 16, true>(H, 4) : wfrag_bytes_t<float, 32, 16, false>(H, 4);
  }
  return 0;
}

// Waves per workgroup of the forward attention kernels of a shape.
int fwd_state_waves(const KernelShape& ks) { return ks.bf16 && ks.m == 128 ? 8 : 4; }

// Workgroups of the forward state pre-pass that run on one CU at a time, from
// the waves per SIMD its launch attributes fix.
int fwd_state_wgs_per_cu(const KernelShape& ks) {
  const int per_simd = state_waves_per_eu(ks.d, ks.nonstationary, fwd_state_waves(ks));
  const int wg_per_simd = fwd_state_waves(ks) / 4;
  return per_simd >= wg_per_simd ? per_simd / wg_per_simd : 1;
}

size_t fwd_state_floats(const KernelShape& ks) {
  const int fw = (ks.m == 64) ? 16 : 32;
  const int nw = ks.m / fw;
  const int fc = 2 * (fw / 16);
  return (size_t)nw * fc * (ks.d / 16 + 1) * WAVE * 4;
}

}  // namespace flex
