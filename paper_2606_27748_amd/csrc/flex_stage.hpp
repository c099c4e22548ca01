// Chunk staging: the raw rows of one 64-token chunk are fetched from HBM once
// per workgroup into registers (16 bytes per load, coalesced), one chunk
// ahead of the computation, then written to LDS where every wave reads the
// operand fragments it needs.  This hides the global-memory latency behind a
// whole chunk of work and removes the redundant per-wave reads.
#pragma once
#include "flex_common.hpp"

namespace flex {

// A window of consecutive rows of a row-major matrix as a raw buffer resource
// (CDNA descriptor word 3): accesses past its last row read zero and drop
// their stores, so ragged chunks need neither a mask nor a branch.  The base
// and the extent are uniform across the workgroup (scalar registers); a
// lane's byte offset into the window does not change from chunk to chunk.
// The sweeps are bound by vector issue, and this takes the 64-bit addresses,
// the zeroing selects and the exec-mask branches around ragged rows out of
// their chunk loops (dK/dV at d = 64, m = 128: 1947 to 1753 instructions per
// chunk).  Before and after, us per pass: d = 64, m = 128 training step (B*H =
// 32, N = 8192) 500 to 480, d = 128, m = 256 2813 to 2626, distillation 250 to
// 232, non-causal m = 64 forward (B*H = 128, N = 16384) 279 to 263.
constexpr int BUF_FLAGS = 0x00020000;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
struct RowBuf {
  __amdgpu_buffer_rsrc_t rs;
  // rows tok0 .. min(n, tok0 + nrows) - 1 of `base` (row_elems elements each); n > tok0
  template <class E>
  __device__ __forceinline__ RowBuf(const E* base, int row_elems, int tok0, int n, int nrows) {
    const int rows = n - tok0 < nrows ? n - tok0 : nrows;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<E*>(base) + (size_t)tok0 * row_elems, 0,
                                           rows * row_elems * (int)sizeof(E), BUF_FLAGS);
  }
  __device__ __forceinline__ uint4 load16(int off) const {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
  }
  __device__ __forceinline__ f32x4 load_f4(int off) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
  }
  __device__ __forceinline__ float load_f1(int off) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
  }
  __device__ __forceinline__ float2 load_f2(int off) const {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
  }
  __device__ __forceinline__ void store16(int off, uint4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, off, 0, 0);
  }
  __device__ __forceinline__ void store_f4(int off, f32x4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, off, 0, 0);
  }
  __device__ __forceinline__ void store_f2(int off, float2 v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rs, off, 0, 0);
  }
  __device__ __forceinline__ void store_f1(int off, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), rs, off, 0, 0);
  }
  // four consecutive values of a row in the io dtype
  __device__ __forceinline__ void store_io4(const u16*, int off, const f32x4& v) const {
    const bf16x4 b = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, b), rs, off, 0, 0);
  }
  __device__ __forceinline__ void store_io4(const float*, int off, const f32x4& v) const { store_f4(off, v); }
};

// Row-major staging of a [64 x COLS] io-typed block with a padded row.
template <class IO, int COLS, int NT, int ROWS = CHUNK>
struct RowStage {
  static constexpr int VEC = 16 / sizeof(IO);           // elements per 16-byte vector
  static constexpr int VPR = COLS / VEC;                 // vectors per row
  static constexpr int NV = ROWS * VPR;                  // vectors per chunk
  static constexpr int PER = (NV + NT - 1) / NT;         // vectors per thread
  static constexpr int LD = COLS + VEC;                  // LDS row stride (elements), keeps 16 B alignment
  static constexpr int LDS_ELEMS = ROWS * LD;
  uint4 r[PER];

  // the stage's thread index (a workgroup of 2 NT threads has two stages)
  static __device__ __forceinline__ int tid() { return (int)(threadIdx.x % NT); }

  // rows: this (b,h) slice's [N, COLS] rows; rows at or beyond n (and the
  // vectors of threads past the chunk) read as zero.  n > tok0.  The chunk's
  // rows are consecutive in memory, so vector v sits 16 v bytes into it: one
  // lane offset for every chunk, and no branch or select on the destination
  // registers, which would make the compiler wait for each load right away.
  __device__ __forceinline__ void fetch(const IO* __restrict__ rows, int tok0, int n) {
    const RowBuf b(rows, COLS, tok0, n, ROWS);
#pragma unroll
    for (int i = 0; i < PER; ++i) r[i] = b.load16((tid() + i * NT) * 16);
  }
  __device__ __forceinline__ uint4 vec(int i) const { return r[i]; }
  // whether vector index v (of thread tid()) is part of the chunk
  static __device__ __forceinline__ bool mine(int v) { return NV % NT == 0 || v < NV; }
  __device__ __forceinline__ void store(IO* lds) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int v = tid() + i * NT;
      if (mine(v)) {
        const int t = v / VPR, c = v % VPR;
        *reinterpret_cast<uint4*>(lds + t * LD + c * VEC) = vec(i);
      }
    }
  }
  // Squared norms are summed in fp32 for bf16 rows and in float64 for fp32
  // rows (the fp32 path's norm factor is formed in float64).
  typedef typename SsqType<IO>::type Ssq;
  // store, plus the squared norm of every row into ssq[ROWS] (the VPR vectors
  // of a row sit in VPR consecutive lanes: summed with lane shuffles)
  __device__ __forceinline__ void store(IO* lds, Ssq* ssq) const {
    store(lds, ssq, [](int, Ssq s) { return s; });
  }
  // store, plus f(row, squared norm of the row) into out[ROWS]
  template <class OUT, class F>
  __device__ __forceinline__ void store(IO* lds, OUT* out, F f) const {
    store_idx(lds, out, [&](int, int t, Ssq s) { return f(t, s); });
  }
  // as store, with f also given the index i < PER of the thread's vector
  template <class OUT, class F>
  __device__ __forceinline__ void store_idx(IO* lds, OUT* out, F f) const {
    static_assert(NT % VPR == 0 && VPR <= WAVE, "a row's vectors must share a wave");
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int v = tid() + i * NT;
      Ssq s = 0;
      if (mine(v)) {
        const int t = v / VPR, c = v % VPR;
        const uint4 x = vec(i);
        *reinterpret_cast<uint4*>(lds + t * LD + c * VEC) = x;
        const IO* e = reinterpret_cast<const IO*>(&x);
#pragma unroll
        for (int j = 0; j < VEC; ++j) { const Ssq y = io_to_float(e[j]); s += y * y; }
      }
      if constexpr (sizeof(Ssq) == 4) {
        s = lane_sum<VPR>(s);
      } else {
#pragma unroll
        for (int o = 1; o < VPR; o <<= 1) s += __shfl_xor(s, o);
      }
      if (mine(v) && v % VPR == 0) out[v / VPR] = f(i, v / VPR, s);
    }
  }
};

// Operand fragment of 8 consecutive columns [c0, c0+8) of LDS row `row`.
__device__ __forceinline__ void lds_row8(Frag<__bf16>& f, const u16* row, int c0) {
  f.v = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(row + c0));
}
__device__ __forceinline__ void lds_row8(Frag<float>& f, const float* row, int c0) {
  const float4 a = *reinterpret_cast<const float4*>(row + c0);
  const float4 b = *reinterpret_cast<const float4*>(row + c0 + 4);
  f.v[0] = a.x; f.v[1] = a.y; f.v[2] = a.z; f.v[3] = a.w;
  f.v[4] = b.x; f.v[5] = b.y; f.v[6] = b.z; f.v[7] = b.w;
}

// fp32 path: one projection tile on the FP64 matrix cores (operand layouts in
// FreqSlice<float>).  ROWS_AS_TOKENS = false: the tile holds frequencies 4g+i
// (rows) x token r (cols), as the bf16 tile of project_tile_lds; true: tokens
// 4g+i x frequency r, as project_rows_lds (the X rows are then permuted so
// that accumulator slot i of lane group g is token 4g + i).
template <int D, int FW, bool NS, int LD, bool ROWS_AS_TOKENS>
__device__ __forceinline__ void project_f64(const FreqSlice<float, D, FW, NS>& fs, const float* X, int tt,
                                            f64x4 (&p)[FreqSlice<float, D, FW, NS>::PR]) {
  typedef FreqSlice<float, D, FW, NS> FS;
  const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  const float* xr = X + (tt * 16 + (ROWS_AS_TOKENS ? f64_tile_row(r) : r)) * LD;
#pragma unroll
  for (int pr = 0; pr < FS::PR; ++pr) p[pr] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < FS::KS; ++ks) {
    const double x = xr[4 * ks + g];
#pragma unroll
    for (int pr = 0; pr < FS::PR; ++pr)
      p[pr] = ROWS_AS_TOKENS ? __builtin_amdgcn_mfma_f64_16x16x4f64(x, fs.wr[pr][ks], p[pr], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f64_16x16x4f64(fs.wt[pr][ks], x, p[pr], 0, 0, 0);
  }
}

// Projection of one 16-token tile (rows staged in LDS, row stride LD) onto a
// wave's frequency slice, plus the squared row norm (summed over lane groups).
template <class T, int D, int FW, bool NS, int LD, class S>
__device__ __forceinline__ void project_tile_lds(const FreqSlice<T, D, FW, NS>& fs,
                                                 const typename Io<T>::type* X, const S* ssq_rows,
                                                 int tt, ProjT<T> (&p)[FreqSlice<T, D, FW, NS>::PR],
                                                 S& ssq) {
  typedef FreqSlice<T, D, FW, NS> FS;
  const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  if constexpr (!IsBf16<T>::value) {
    project_f64<D, FW, NS, LD, false>(fs, X, tt, p);
  } else {
    const typename Io<T>::type* row = X + (tt * 16 + r) * LD;
#pragma unroll
    for (int pr = 0; pr < FS::PR; ++pr) p[pr] = zero4();
#pragma unroll
    for (int ks = 0; ks < FS::KD; ++ks) {
      Frag<T> x;
      lds_row8(x, row, ks * 32 + 8 * g);
#pragma unroll
      for (int pr = 0; pr < FS::PR; ++pr)
#pragma unroll
        for (int sp = 0; sp < FS::NSPLIT; ++sp) mma(p[pr], fs.w[sp][pr][ks], x);
    }
  }
  ssq = ssq_rows[tt * 16 + r];
}

template <class T, int D, int FW, int NW, bool NS, int CH_ = CHUNK>
struct Shape {
  static constexpr int CH = CH_;            // tokens per chunk
  static constexpr int TT = CH / 16;        // token tiles per chunk
  static constexpr int M = FW * NW;
  static constexpr int FT = FW / 16;        // frequency tiles per wave
  static constexpr int FC = 2 * FT;         // feature tiles per wave
  static constexpr int DV = D;
  static constexpr int DVT = DV / 16;       // value tiles
  static constexpr int DVT1 = DVT + 1;      // + the normaliser tile
  static constexpr int KT = CH / 32;        // k-steps over the tokens of a chunk
  static constexpr int PR = NS ? 2 * FT : FT;
  static constexpr int NT = NW * WAVE;      // threads per workgroup
  // fp32 floats of one wave's state, one (b,h,segment) block of the workspace
  static constexpr int WAVE_STATE = FC * DVT1 * WAVE * 4;
  static constexpr int STATE = NW * WAVE_STATE;
  // LDS row strides (elements); multiples of 4 keep 8/16-byte alignment
  static constexpr int TPAD = CH + 4;
  static constexpr int RPAD = DVT1 * 16 + 4;
};

// Fragment of ones: as the value operand it appends the ones column of
// [V | 1] that produces the normaliser, in all 16 columns of its tile alike
// (so every lane of a readout holds its token's denominator).
template <class T>
__device__ __forceinline__ Frag<T> ones_all() {
  Frag<T> f;
#pragma unroll
  for (int j = 0; j < 8; ++j) f.set(j, 1.0f);
  return f;
}

// Operand fragment over the chunk's tokens from a token-contiguous LDS row:
// slots j<4 take tokens 32ks+4g+j, slots j>=4 tokens 32ks+16+4g+j-4.  This is
// the token order of a pair of accumulator tiles (see pair_tiles).
template <class T>
__device__ __forceinline__ Frag<T> lds_tok_frag(const T* row, int ks) {
  const int g = (threadIdx.x % WAVE) / 16;
  Frag<T> f;
  const T* a = row + 32 * ks + 4 * g;
  const T* b = a + 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) { f.set(j, (float)a[j]); f.set(4 + j, (float)b[j]); }
  return f;
}
template <>
__device__ __forceinline__ Frag<__bf16> lds_tok_frag<__bf16>(const __bf16* row, int ks) {
  const int g = (threadIdx.x % WAVE) / 16;
  const __bf16* a = row + 32 * ks + 4 * g;
  bf16x4 lo = *reinterpret_cast<const bf16x4*>(a);
  bf16x4 hi = *reinterpret_cast<const bf16x4*>(a + 16);
  Frag<__bf16> f;
  f.v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return f;
}

// Two accumulator tiles whose rows are consecutive 16-blocks of a contraction
// index, as one operand fragment (slots 0..3 from the first, 4..7 from the second).
template <class T>
__device__ __forceinline__ Frag<T> pair_tiles(const f32x4& a, const f32x4& b) {
  Frag<T> f;
#pragma unroll
  for (int i = 0; i < 4; ++i) { f.set(i, a[i]); f.set(4 + i, b[i]); }
  return f;
}

// Two accumulator tiles as one operand fragment split into a high and a low
// part (bf16 hi + lo carries about 16 significant bits; fp32 keeps the value).
template <class T>
__device__ __forceinline__ void split_pair(const f32x4& a, const f32x4& b, Frag<T>& hi, Frag<T>& lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi.set(i, a[i]);
    hi.set(4 + i, b[i]);
    lo.set(i, a[i] - hi.get(i));
    lo.set(4 + i, b[i] - hi.get(4 + i));
  }
}

// A low part x - hi, or a sum of low parts, as it is added to the high one: where x
// overflows the operand type, hi is infinite and the low part infinite or NaN, and
// one med3 makes it finite (a NaN gives the lower limit), so that the sum stays
// infinite, as with hi alone.  The low part of a finite x is at most 2^-9 |x|, and
// sums of a chunk's stay below the limits unless x overflows.
__device__ __forceinline__ float finite_low(float lo) { return __builtin_amdgcn_fmed3f(lo, -1e37f, 1e37f); }

// Projection of one 16-token tile with the tokens as rows: p[pr] holds rows =
// tokens tt*16 + 4g + i and cols = frequency (lane % 16) of projection tile
// pr.  The operands of project_tile_lds are swapped (the register layouts of
// the two MFMA operands are the same), so the frequency fragments are shared.
template <class T, int D, int FW, bool NS, int LD>
__device__ __forceinline__ void project_rows_lds(const FreqSlice<T, D, FW, NS>& fs,
                                                 const typename Io<T>::type* X, int tt,
                                                 ProjT<T> (&p)[FreqSlice<T, D, FW, NS>::PR]) {
  typedef FreqSlice<T, D, FW, NS> FS;
  if constexpr (!IsBf16<T>::value) {
    project_f64<D, FW, NS, LD, true>(fs, X, tt, p);
  } else {
    const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
    const typename Io<T>::type* row = X + (tt * 16 + r) * LD;
#pragma unroll
    for (int pr = 0; pr < FS::PR; ++pr) p[pr] = zero4();
#pragma unroll
    for (int ks = 0; ks < FS::KD; ++ks) {
      Frag<T> x;
      lds_row8(x, row, ks * 32 + 8 * g);
#pragma unroll
      for (int pr = 0; pr < FS::PR; ++pr)
#pragma unroll
        for (int sp = 0; sp < FS::NSPLIT; ++sp) mma(p[pr], x, fs.w[sp][pr][ks]);
    }
  }
}

// Features of a wave's frequency slice for the 32 tokens of k-step ks, with
// the tokens as the contraction index: out[2ft] (cos-type) and out[2ft+1]
// (sin-type) have cols = the feature (lane % 16) and k = tokens in the order
// of pair_tiles / lds_tok_frag.  sc[t] is the per-token scale (0 for tokens
// past the end).  Used where a feature map only enters contractions over
// tokens (state sums), which then need no transpose through LDS.  fv: as in
// features (slice frequencies ft*16 + lane%16 >= fv give zero features).
template <class T, int D, int FW, bool NS, int LD>
__device__ __forceinline__ void feature_frags_rows(const FreqSlice<T, D, FW, NS>& fs,
                                                   const typename Io<T>::type* X, const float* sc,
                                                   int ks, Frag<T> (&out)[2 * (FW / 16)], int fv = FW) {
  typedef FreqSlice<T, D, FW, NS> FS;
  constexpr int FT = FW / 16;
  const int g = (threadIdx.x % WAVE) / 16;
  f32x4 fc[2][FT], fsn[2][FT];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int tt = 2 * ks + hh;
    ProjT<T> p[FS::PR];
    project_rows_lds<T, D, FW, NS, LD>(fs, X, tt, p);
    const float4 s4 = *reinterpret_cast<const float4*>(sc + tt * 16 + 4 * g);
    const float sv[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float s1, c1;
        sincos_rev(p[ft][i], s1, c1);
        const float m = NS ? sv[i] * cos_rev(p[FT + ft][i]) : sv[i];
        fc[hh][ft][i] = c1 * m;
        fsn[hh][ft][i] = s1 * m;
      }
  }
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    out[2 * ft] = pair_tiles<T>(fc[0][ft], fc[1][ft]);
    out[2 * ft + 1] = pair_tiles<T>(fsn[0][ft], fsn[1][ft]);
  }
  if (fv < FW) {   // this lane's frequency is slice frequency ft*16 + lane % 16
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
      if (ft * 16 + (int)(threadIdx.x % 16) >= fv) { out[2 * ft].zero(); out[2 * ft + 1].zero(); }
  }
}

// ---------------------------------------------------------------------------
// Transposes through LDS with the gfx950 transpose load.  An accumulator tile
// holds column n = lane % 16 and rows m = 4g + i (g = lane / 16); written as
// bf16 into an [n][m]-major block it is one 8-byte store per lane.  Reading
// that block back with ds_read_b64_tr_b16 gives an operand whose lane is m and
// whose k index is n: within each group of 16 lanes, slot j of lane i receives
// element i % 4 of the 4-element row addressed by lane 4j + i / 4, so lane
// (g, i) addresses row kb + i / 4, columns m0 + 4 (i % 4) .. + 3, and receives
// column m0 + i of rows kb .. kb + 3.  The fp32 operand type keeps plain
// element-wise accesses of the same layouts.
// ---------------------------------------------------------------------------
typedef short tr_v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) tr_v4i16 lds_tr_v4i16;

// Rows 4g..4g+3 of an accumulator tile (values v) into L[n][m0 + 4g + i],
// n = n0 + lane % 16.
template <class T>
__device__ __forceinline__ void store_tile_nm(T* L, int ld, int n0, int m0, const f32x4& v) {
  const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  T* o = L + (n0 + r) * ld + m0 + 4 * g;
  if constexpr (IsBf16<T>::value) {
    const bf16x4 b = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    *reinterpret_cast<bf16x4*>(o) = b;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = v[i];
  }
}

// The two halves of an operand fragment (slots 0..3 and 4..7, each four rows
// 4g..4g+3 of one tile) into L[n][m0a + 4g + i] and L[n][m0b + 4g + i].
template <class T>
__device__ __forceinline__ void store_frag_nm(T* L, int ld, int n0, int m0a, int m0b, const Frag<T>& f) {
  const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  T* row = L + (n0 + r) * ld + 4 * g;
  if constexpr (IsBf16<T>::value) {
    const uint4 w = __builtin_bit_cast(uint4, f.v);
    *reinterpret_cast<uint2*>(row + m0a) = make_uint2(w.x, w.y);
    *reinterpret_cast<uint2*>(row + m0b) = make_uint2(w.z, w.w);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) { row[m0a + i] = f.raw(i); row[m0b + i] = f.raw(4 + i); }
  }
}

// Operand fragment stored by store_frag_nm, read back in the same layout:
// lane row n0 + lane % 16, slots 0..3 from columns m0a + 4g .. + 3, slots
// 4..7 from m0b + 4g .. + 3.
template <class T>
__device__ __forceinline__ Frag<T> load_frag_nm(const T* L, int ld, int n0, int m0a, int m0b) {
  const int l = threadIdx.x % WAVE, r = l % 16, g = l / 16;
  const T* row = L + (n0 + r) * ld + 4 * g;
  Frag<T> f;
  if constexpr (IsBf16<T>::value) {
    const uint2 a = *reinterpret_cast<const uint2*>(row + m0a);
    const uint2 b = *reinterpret_cast<const uint2*>(row + m0b);
    f.v = __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) { f.set(i, row[m0a + i]); f.set(4 + i, row[m0b + i]); }
  }
  return f;
}

// Operand fragment with lane m = m0 + lane % 16 and k slots 0..3 = rows
// kb0 .. kb0+3, slots 4..7 = rows kb1 .. kb1+3 of an [k][m]-major block
// (kb0, kb1 may differ between lane groups).
template <class T>
__device__ __forceinline__ Frag<T> lds_tr_frag(const T* L, int ld, int kb0, int kb1, int m0) {
  const int i = (threadIdx.x % WAVE) % 16;
  Frag<T> f;
  if constexpr (IsBf16<T>::value) {
    const int off = (i / 4) * ld + m0 + 4 * (i % 4);
    const tr_v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_v4i16*)(L + kb0 * ld + off));
    const tr_v4i16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_v4i16*)(L + kb1 * ld + off));
    f.v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f.set(j, L[(kb0 + j) * ld + m0 + i]);
      f.set(4 + j, L[(kb1 + j) * ld + m0 + i]);
    }
  }
  return f;
}

// One wave's operand fragment in LDS as it is held, 8 slots per lane (fp32:
// the lane groups 32 bytes further apart, so that the transposed reads of tr()
// fall into different banks).
template <class T>
struct FragLds {
  static constexpr int PAD = IsBf16<T>::value ? 0 : 8;   // elements per lane group
  __attribute__((aligned(16))) T v[WAVE * 8 + 4 * PAD];
  static __device__ __forceinline__ int at(int l) { return l * 8 + l / 16 * PAD; }
  __device__ __forceinline__ void put(int l, const Frag<T>& f) { *reinterpret_cast<decltype(f.v)*>(v + at(l)) = f.v; }
  __device__ __forceinline__ Frag<T> get(int l) const {
    Frag<T> f;
    f.v = *reinterpret_cast<const decltype(f.v)*>(v + at(l));
    return f;
  }
};
template <>
__device__ __forceinline__ void FragLds<float>::put(int l, const Frag<float>& f) {
  float4* o = reinterpret_cast<float4*>(v + at(l));
  o[0] = make_float4(f.v[0], f.v[1], f.v[2], f.v[3]);
  o[1] = make_float4(f.v[4], f.v[5], f.v[6], f.v[7]);
}
template <>
__device__ __forceinline__ Frag<float> FragLds<float>::get(int l) const {
  Frag<float> f;
  lds_row8(f, v + at(l), 0);
  return f;
}

// The transpose load from two fragments in LDS: f0 holds columns (lane % 16)
// 0..15, f1 16..31, its slots 4 half + (0..3) the rows 4g + (0..3) of one
// tile.  The result has lane m = row and k slots 0..3 = columns 4g .. 4g+3
// (f0), 4..7 = columns 16 + 4g .. (f1).
template <class T>
__device__ __forceinline__ Frag<T> tr_of_frags(const FragLds<T>& f0, const FragLds<T>& f1, int half) {
  const int l = threadIdx.x % WAVE, i = l % 16, g = l / 16;
  Frag<T> f;
  if constexpr (IsBf16<T>::value) {
    // lane i of a group addresses column 4g + i/4, rows 4 (i % 4) .. + 3
    const int at = FragLds<T>::at(16 * (i % 4) + 4 * g + i / 4) + 4 * half;
    const tr_v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_v4i16*)(f0.v + at));
    const tr_v4i16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_v4i16*)(f1.v + at));
    f.v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  } else {
    // lane i is row i: slot i % 4 of the fragments of lanes 16 (i / 4) + column
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int at = FragLds<T>::at(16 * (i / 4) + 4 * g + j) + 4 * half + i % 4;
      f.set(j, f0.v[at]);
      f.set(4 + j, f1.v[at]);
    }
  }
  return f;
}

}  // namespace flex
