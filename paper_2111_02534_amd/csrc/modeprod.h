// Mode-product tiles (device bodies): Y = L X + X R (+ epilogue) on the FP64 and
// FP32 matrix cores, see ModeProd in kernels.h.  Included by HIP translation
// units only.
//
// FP64 and FP32 matrix instructions run on the vector ALUs' own multipliers: a
// SIMD that issues a VALU instruction issues no product in that slot.  So the K
// loop is written to need none:
//  * The constant operands never touch LDS.  They are stored in MFMA fragment
//    order (mp_fragments), padded with zeros, and a wave reads the fragments of
//    its own rows or columns from the L2 with 16-byte loads, one K group (two
//    FP64 or four FP32 K steps) ahead of their use: uniform base, constant lane
//    offset.
//  * The vector's chunk goes through registers into LDS in 16-byte pieces, again
//    from a uniform base with constant lane offsets, the next chunk's loads in
//    flight while the current one is multiplied, two buffers and one barrier per
//    chunk.  Clamping, zero filling and unaligned rows have a path of their own,
//    which only the last chunk of a ragged K range or an unaligned vector takes.
//  * A K group's k are dealt to the four lane groups of the instruction so
//    that a lane's two (four) k are neighbours: lane group g owns k = KU g + u
//    of the group in K step u.  The rows-by-k operand (X in X R) is then read as
//    one ds_read_b128 per K group.  For the k-by-columns operand (X in L X) the
//    columns are dealt likewise: block b of a pair takes columns 2 l + b of 32, so
//    a read gives both blocks' operands and a lane's two outputs are
//    neighbours in memory.
#pragma once

#include <type_traits>

#include "device_bodies.h"

namespace tp3b {

template <typename T>
struct MpVec;
template <>
struct MpVec<double> {
  static constexpr int KU = 2;  // K steps per fragment piece, elements per piece
  typedef double2 piece;
  typedef double2 pair;
};
template <>
struct MpVec<float> {
  static constexpr int KU = 4;
  typedef float4 piece;
  typedef float2 pair;
};

// element u of a piece (u a constant after unrolling)
template <typename T>
__device__ __forceinline__ T mp_at(const typename MpVec<T>::piece& p, int u) {
  if constexpr (sizeof(T) == 8) return u == 0 ? p.x : p.y;
  else return u == 0 ? p.x : (u == 1 ? p.y : (u == 2 ? p.z : p.w));
}

// Tile shapes: SK waves split every K chunk (each takes its own K groups and
// computes the whole wave tile), WM x WN waves tile the output, each with
// BM x BN MFMA blocks.
template <typename T, int BM, int BN, int WM, int WN, int SK>
struct MpTile {
  static constexpr int KU = MpVec<T>::KU;
  static constexpr int KG = 4 * KU;       // k per K group
  static constexpr int KC = 2 * KG;       // k per wave and chunk (two K groups)
  static constexpr int KT = KC * SK;      // k per chunk
  static constexpr int NW = WM * WN * SK, NT = 64 * NW;
  static constexpr int TM = 16 * BM * WM, TN = 16 * BN * WN;
  // left chunk: rows of TN entries; FP32 rows are padded by 32 bytes, so that
  // rows four apart (read together) start half the banks apart
  static constexpr int LDL = TN + (sizeof(T) == 4 ? 8 : 0);
  static constexpr int SPR = KT / KU;     // pieces per row of the right chunk
  static constexpr int SZL = KT * LDL, SZR = TM * KT;
  static constexpr int SZ = SZL > SZR ? SZL : SZR;
  static constexpr int PL = KT * TN / KU / NT, PR = TM * KT / KU / NT;  // pieces per thread
  static constexpr int PM = PL > PR ? PL : PR;
  static_assert(BN % 2 == 0, "column blocks come in pairs");
  static_assert(PL * NT * KU == KT * TN && PR * NT * KU == TM * KT, "chunk not divisible among the threads");
  static constexpr int SUM = SK > 1 ? SK * TM * TN : 1;
  struct Smem {
    union {
      __attribute__((aligned(16))) T buf[2][SZ];
      T red[SUM];
    };
  };
  // place of piece s of row r in the right chunk: the sixteen rows read
  // together fall on different banks
  static __device__ __forceinline__ int slot(int r, int s) {
    return r * SPR + (s ^ (SPR >= 16 ? (r & 15) : ((r >> 1) & (SPR - 1))));
  }
};

// Sizes of the fragment arrays: rows padded to 32, k to 16.
__host__ __device__ inline int mp_pad_rows(int n) { return (n + 31) / 32 * 32; }
__host__ __device__ inline int mp_pad_k(int n) { return (n + 15) / 16 * 16; }

// Buffer loads: a uniform 64-bit base and byte count in scalar registers and a
// 32-bit byte offset per lane, so that stepping through a matrix costs no vector
// instruction; what lies at or past the count reads as zero.
typedef uint32_t mp_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t mp_u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int64_t mp_uniform(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t mp_buffer(const char* p, int64_t bytes) {
  const int64_t n = bytes < 0 ? 0 : (bytes < 0xffffffffll ? bytes : 0xffffffffll);
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)(uint32_t)n, 0x00027000);
}
template <typename P>
__device__ __forceinline__ P mp_load(__amdgpu_buffer_rsrc_t b, uint32_t off) {
  if constexpr (sizeof(P) == 16) return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
  else if constexpr (sizeof(P) == 8) return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0));
  else return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0));
}

// The two phases of the K loop: L X, then X R.
struct MpLeft { static constexpr bool left = true; };
struct MpRight { static constexpr bool left = false; };

// How the vector is read: in whole pieces (16-byte aligned rows, a multiple of a
// piece long), element by element, or element by element with 64-bit offsets (left
// products whose chunks reach further than a buffer load's 32-bit offset).
enum MpRead { MP_WHOLE, MP_ELEMENTS, MP_FAR };

// Output tile w of the product `a`.  MODE (MpMode): what the product does to its
// operand or result besides:
//   fold    the operand is X[k] + X[k'] (item 0) or X[k] - X[k'] (item 1) with
//           k' the mirror of k, formed while a chunk is put into LDS;
//   unfold  two products over K, of the even and of the odd operand, whose sum
//           and difference go to an output and its mirror.
template <typename T, int BM, int BN, int WM, int WN, int SK, int READ, int MODE>
__device__ __forceinline__ void mp_tile_w(const ModeProd<T>& a, int64_t w,
                                          typename MpTile<T, BM, BN, WM, WN, SK>::Smem& sm) {
  typedef MpTile<T, BM, BN, WM, WN, SK> G;
  typedef typename MpVec<T>::piece piece;
  typedef typename MpVec<T>::pair pair;
  typedef typename Mma<T>::acc_t acc_t;
  constexpr int KU = G::KU, BF = BM > BN ? BM : BN;
  constexpr bool FOLD = MODE == MP_FOLD_L || MODE == MP_FOLD_R, UNFOLD = MODE == MP_UNFOLD_L || MODE == MP_UNFOLD_R;
  constexpr bool LEFT_ONLY = MODE == MP_FOLD_L || MODE == MP_UNFOLD_L || READ == MP_FAR;
  constexpr bool RIGHT_ONLY = MODE == MP_FOLD_R || MODE == MP_UNFOLD_R;
  static_assert(READ != MP_FAR || MODE == MP_PLAIN, "only plain products have rows this long");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int sk = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  const int M = __builtin_amdgcn_readfirstlane(a.M), Nc = __builtin_amdgcn_readfirstlane(a.Nc);
  const int full = __builtin_amdgcn_readfirstlane(a.full);
  const int64_t rs = mp_uniform(a.rs), rsy = MODE == MP_PLAIN ? rs : mp_uniform(a.rsy);
  const int tiles_n = (Nc + G::TN - 1) / G::TN;
  const int64_t tiles = (int64_t)((M + G::TM - 1) / G::TM) * tiles_n;
  const int64_t q = w / tiles;
  const int t = __builtin_amdgcn_readfirstlane((int)(w - q * tiles));
  const int i0 = (t / tiles_n) * G::TM, j0 = (t % tiles_n) * G::TN;
  const int64_t vec = q / a.per_vec;
  const int item = __builtin_amdgcn_readfirstlane((int)(q - vec * a.per_vec));
  const T* __restrict__ X = (const T*)mp_uniform((int64_t)(a.X + vec * a.ldx + (FOLD ? 0 : item * a.bstride)));
  T* __restrict__ Y = (T*)mp_uniform((int64_t)(a.Y + vec * a.ldy + item * a.bstride));

  const int kx = mp_pad_k(M) / G::KG, ky = mp_pad_k(Nc) / G::KG;          // K groups
  const int bx = mp_pad_rows(M) >> 4, by = mp_pad_rows(Nc) >> 4;          // blocks of 16 rows or columns
  const bool hasL = MODE == MP_PLAIN ? a.LF != nullptr : LEFT_ONLY, hasR = MODE == MP_PLAIN ? a.RF != nullptr : RIGHT_ONLY;
  const int nL = __builtin_amdgcn_readfirstlane(hasL ? (M + G::KT - 1) / G::KT : 0);
  const int nR = __builtin_amdgcn_readfirstlane(hasR ? (Nc + G::KT - 1) / G::KT : 0);
  const int nch = UNFOLD ? 2 * (nL + nR) : nL + nR;
  // fragments of this wave's blocks (byte offset inside a K group); blocks past
  // the matrix read its last one (their outputs are not stored)
  const char* LFi = (const char*)mp_uniform((int64_t)(a.LF + (FOLD ? item * a.fq : 0)));
  const char* RFi = (const char*)mp_uniform((int64_t)(a.RF + (FOLD ? item * a.fq : 0)));
  uint32_t fl[BM], fr[BN];
#pragma unroll
  for (int b = 0; b < BM; ++b) fl[b] = (uint32_t)(min((i0 >> 4) + wm * BM + b, bx - 1) * 64 + lane) * 16;
#pragma unroll
  for (int b = 0; b < BN; ++b) fr[b] = (uint32_t)(min((j0 >> 4) + wn * BN + b, by - 1) * 64 + lane) * 16;

  acc_t acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // This thread's piece s of a left chunk is row rl + s DL, columns cl .. of the
  // tile's columns; of a right chunk row rr + s DR of the tile's rows, k cr ...
  constexpr int PPR = G::TN / KU;  // pieces per row of a left chunk
  constexpr int DL = G::NT / PPR, DR = G::NT / G::SPR;
  static_assert(DL * PPR == G::NT && DR * G::SPR == G::NT, "pieces are dealt out in whole rows");
  const int rl = tid / PPR, cl = (tid % PPR) * KU, rr = tid / G::SPR, cr = (tid % G::SPR) * KU;
  // Byte offsets of the pieces from the first row of a left chunk, from the first
  // entry of a right one (32-bit: the launcher keeps to tiles whose rows reach no
  // further).  Rows past the vector read as zero; columns past a row's end read
  // the next row, and go to outputs that are not stored.
  constexpr uint32_t ES = sizeof(T);
  const uint32_t rsb = (uint32_t)(rs * ES);
  uint32_t vl[G::PL], vr[G::PR];
#pragma unroll
  for (int s = 0; s < G::PL; ++s) vl[s] = (rl + s * DL) * rsb + (uint32_t)(j0 + cl) * ES;
#pragma unroll
  for (int s = 0; s < G::PR; ++s) vr[s] = (rr + s * DR) * rsb + (uint32_t)cr * ES;
  // bytes of the vector
  const int64_t extent = ((MODE == MP_FOLD_L ? full - 1 : M - 1) * rs + (MODE == MP_FOLD_R ? full : Nc)) * ES;
  // chunk of its operand that chunk c of the loop takes
  auto place = [&](auto ph, int c) { return UNFOLD ? (c < nch / 2 ? c : c - nch / 2) : (ph.left ? c : c - nL); };

  piece raw[G::PM], mir[FOLD ? G::PM : 1];
  auto fetch = [&](__amdgpu_buffer_rsrc_t b, uint32_t off) -> piece {
    if constexpr (READ == MP_WHOLE) {
      return mp_load<piece>(b, off);
    } else {
      T v[KU];
#pragma unroll
      for (int u = 0; u < KU; ++u) v[u] = mp_load<T>(b, off + u * ES);
      return __builtin_bit_cast(piece, v);
    }
  };
  auto load = [&](auto ph, int c) {
    c = min(c, nch - 1);
    const int k0 = place(ph, c) * G::KT;
    // unfold: the odd operand, M rows or a half row on
    const int64_t odd = UNFOLD && c >= nch / 2 ? a.oddx : 0;
    const int64_t at = (odd + (ph.left ? k0 * rs : i0 * rs + k0)) * ES;
    const __amdgpu_buffer_rsrc_t b = mp_buffer((const char*)X + at, odd * ES + extent - at);
    constexpr int P = ph.left ? G::PL : G::PR;
    if constexpr (READ == MP_FAR && ph.left) {
      // (as the buffer reads: rows past the vector are zero)
#pragma unroll
      for (int s = 0; s < P; ++s) {
        const int64_t e = (k0 + rl + s * DL) * rs + j0 + cl;
        T v[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) v[u] = (e + u) * (int64_t)ES < extent ? X[e + u] : T(0);
        raw[s] = __builtin_bit_cast(piece, v);
      }
    } else {
#pragma unroll
      for (int s = 0; s < P; ++s) raw[s] = fetch(b, ph.left ? vl[s % G::PL] : vr[s % G::PR]);
    }
    if constexpr (FOLD) {
      // the mirrors: rows full-1-k, or columns full-1-k in reverse order.  Places
      // before the vector's start (k past the half) wrap to offsets past its end.
      const __amdgpu_buffer_rsrc_t m = mp_buffer((const char*)X, extent);
#pragma unroll
      for (int s = 0; s < P; ++s) {
        if constexpr (ph.left) {
          mir[s] = fetch(m, (uint32_t)(full - 1 - k0 - (rl + s * DL)) * rsb + (uint32_t)(j0 + cl) * ES);
        } else {
          const uint32_t row = (uint32_t)(i0 + rr + s * DR) * rsb;
          const int first = full - KU - k0 - cr;  // mirror of the piece's last k
          if constexpr (READ == MP_WHOLE) {
            mir[s] = fetch(m, row + (uint32_t)first * ES);
          } else {
            // a piece of a short row may start before it: those are k past the half
            T v[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) v[u] = mp_load<T>(m, row + (uint32_t)max(first + u, 0) * ES);
            mir[s] = __builtin_bit_cast(piece, v);
          }
        }
      }
    }
  };
  auto store = [&](auto ph, int c, T* buf) {
    c = min(c, nch - 1);
    constexpr int P = ph.left ? G::PL : G::PR;
    auto at = [&](int s) { return (piece*)(buf + (ph.left ? (rl + s * DL) * G::LDL + cl : G::slot(rr + s * DR, cr / KU) * KU)); };
    const int k0 = place(ph, c) * G::KT;
    if constexpr (FOLD) {
      const T sg = item ? T(-1) : T(1);
#pragma unroll
      for (int s = 0; s < P; ++s) {
        T v[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
          v[u] = mp_at<T>(raw[s], u) + sg * mp_at<T>(mir[s], ph.left ? u : KU - 1 - u);
          // k past the half: zero
          if (k0 + G::KT > (ph.left ? M : Nc))
            v[u] = (ph.left ? k0 + rl + s * DL < M : k0 + cr + u < Nc) ? v[u] : T(0);
        }
        *at(s) = __builtin_bit_cast(piece, v);
      }
    } else if (ph.left || k0 + G::KT <= Nc) {
#pragma unroll
      for (int s = 0; s < P; ++s) *at(s) = raw[s];
    } else {
      // k past the end of a row: zero (the next row was read)
#pragma unroll
      for (int s = 0; s < P; ++s) {
        T v[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) v[u] = k0 + cr + u < Nc ? mp_at<T>(raw[s], u) : T(0);
        *at(s) = __builtin_bit_cast(piece, v);
      }
    }
  };
  // fragments of K group g (0, 1) of this wave in chunk c
  piece f[2][BF];
  const int skg = __builtin_amdgcn_readfirstlane(sk * 2);
  auto loadf = [&](auto ph, int c, int g) {
    c = min(c, nch - 1);
    const int kg = min(place(ph, c) * (G::KT / G::KG) + skg + g, (ph.left ? kx : ky) - 1);
    const int nb = (ph.left ? bx : by) * 1024;
    const int64_t odd = UNFOLD && c >= nch / 2 ? a.fq * ES : 0;
    const __amdgpu_buffer_rsrc_t F = mp_buffer((ph.left ? LFi : RFi) + odd + (int64_t)kg * nb, nb);
    constexpr int B = ph.left ? BM : BN;
#pragma unroll
    for (int b = 0; b < B; ++b) f[g][b] = mp_load<piece>(F, ph.left ? fl[b % BM] : fr[b % BN]);
  };
  // One chunk of phase ph in 2 KU K steps, with the loads of the chunk after it
  // (phase nx).  The LDS operands of a step are read a step (of the right
  // phase: a K group) ahead; the loads and LDS stores are dealt out between
  // the matrix instructions of the first and the last step.
  auto chunk = [&](auto ph, auto nx, int c) {
    const T* buf = sm.buf[c & 1];
    constexpr bool left = ph.left;
    pair xl[2][BN / 2];
    piece xr[2][BM];
    auto read = [&](int t) {  // the operands of step t (left), of K group t (right)
      if constexpr (left) {
        const T* row = buf + (sk * G::KC + KU * lk) * G::LDL + wn * 16 * BN + 2 * lr + ((t / KU) * G::KG + t % KU) * G::LDL;
#pragma unroll
        for (int j = 0; j < BN / 2; ++j) xl[t & 1][j] = *(const pair*)(row + 32 * j);
      } else {
#pragma unroll
        for (int i = 0; i < BM; ++i)
          xr[t][i] = ((const piece*)buf)[G::slot((wm * BM + i) * 16 + lr, sk * (G::KC / KU) + t * 4 + lk)];
      }
    };
    read(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2 * KU; ++t) {
      if (left && t + 1 < 2 * KU) read(t + 1);
      if (!left && t == KU - 1) read(1);
      if (t == 0) {
        loadf(ph, c, 1);
        load(nx, c + 1);
      }
      if (t == KU) loadf(nx, c + 1, 0);
      if (t == 2 * KU - 1) store(nx, c + 1, sm.buf[(c + 1) & 1]);
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) {
          if constexpr (left)
            acc[i][j] = Mma<T>::mma(mp_at<T>(f[t / KU][i], t % KU), (j & 1 ? xl[t & 1][j / 2].y : xl[t & 1][j / 2].x),
                                    acc[i][j]);
          else
            acc[i][j] = Mma<T>::mma(mp_at<T>(xr[t / KU][i], t % KU), mp_at<T>(f[t / KU][j], t % KU), acc[i][j]);
        }
#pragma unroll
      for (int m = 0; m < BM * BN; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // VALU
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global load
        __builtin_amdgcn_sched_group_barrier(0x080, 1, 0);  // LDS
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  };

  auto start = [&](auto ph) {
    load(ph, 0);
    loadf(ph, 0, 0);
    store(ph, 0, sm.buf[0]);
    __syncthreads();
  };
  acc_t even[UNFOLD ? BM : 1][UNFOLD ? BN : 1];
  if constexpr (MODE == MP_PLAIN && !LEFT_ONLY) {
    if (nL) start(MpLeft());
    else start(MpRight());
    int c = 0;
    for (const int e = nR ? nL - 1 : nL; c < e; ++c) chunk(MpLeft(), MpLeft(), c);
    if (nL && nR) {
      chunk(MpLeft(), MpRight(), c);
      ++c;
    }
    for (; c < nch; ++c) chunk(MpRight(), MpRight(), c);
  } else {
    typedef typename std::conditional<LEFT_ONLY, MpLeft, MpRight>::type Ph;
    start(Ph());
    int c = 0;
    if constexpr (UNFOLD) {
      for (; c < nch / 2; ++c) chunk(Ph(), Ph(), c);
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) {
          even[i][j] = acc[i][j];
          acc[i][j] = acc_t{0, 0, 0, 0};
        }
    }
    for (; c < nch; ++c) chunk(Ph(), Ph(), c);
  }

  // epilogue: two neighbouring columns at a time
  const T shift = a.epi == EPI_V ? T(a.shifts ? a.shifts[vec] : 0.0) : T(0);
  const T* Vp = a.V ? a.V + item * a.bstride : nullptr;
  const T* lamR = a.lamR + (FOLD ? item * a.lamRq : 0);
  const T lams = a.epi == EPI_DIV && a.lamItem ? a.lamItem[item] : T(0);
  const bool pairs = (((uintptr_t)X | (uintptr_t)Y | (uintptr_t)Vp | (uintptr_t)(rs * (int64_t)ES) |
                       (uintptr_t)(rsy * (int64_t)ES)) &
                      (2 * ES - 1)) == 0;
  // the entries of the vector and the potential at a pair of outputs
  auto operands = [&](int gi, int gj, pair& x, pair& p) {
    x = p = pair{0, 0};
    if (MODE != MP_PLAIN || a.epi != EPI_V || gi >= M || gj >= Nc) return;
    const int64_t off = (int64_t)gi * rs + gj;
    if (pairs && gj + 1 < Nc) {
      x = *(const pair*)(X + off);
      if (Vp) p = *(const pair*)(Vp + off);
    } else {
      x.x = X[off];
      if (gj + 1 < Nc) x.y = X[off + 1];
      if (Vp) {
        p.x = Vp[off];
        if (gj + 1 < Nc) p.y = Vp[off + 1];
      }
    }
  };
  auto put = [&](int64_t off, bool two, T v0, T v1) {
    if (pairs && two && (off & 1) == 0) {
      *(pair*)(Y + off) = pair{v0, v1};
    } else {
      Y[off] = v0;
      if (two) Y[off + 1] = v1;
    }
  };
  auto emit = [&](int gi, int gj, T v0, T v1, const pair& x, const pair& p) {
    if (gi >= M || gj >= Nc) return;
    const int64_t off = (int64_t)gi * rsy + gj;
    const bool two = gj + 1 < Nc;
    if (MODE == MP_PLAIN && a.epi == EPI_V) {
      v0 += (p.x - shift) * x.x;
      v1 += (p.y - shift) * x.y;
    } else if (a.epi == EPI_DIV) {
      const T l = a.lamL[gi];
      v0 = v0 / (l + lamR[gj] + lams - T(a.sigma));
      if (two) v1 = v1 / (l + lamR[gj + 1] + lams - T(a.sigma));
    }
    if (MODE == MP_PLAIN && a.acc) {
      v0 += Y[off];
      if (two) v1 += Y[off + 1];
    }
    put(off, two, v0, v1);
  };
  // unfold: the sums at (gi, gj), the differences at the mirror
  auto emit2 = [&](int gi, int gj, T e0, T e1, T o0, T o1) {
    if (gi >= M || gj >= Nc) return;
    const bool two = gj + 1 < Nc;
    put((int64_t)gi * rsy + gj, two, e0 + o0, e1 + o1);
    if (MODE == MP_UNFOLD_L) {
      const int g2 = full - 1 - gi;
      if (g2 != gi) put((int64_t)g2 * rsy + gj, two, e0 - o0, e1 - o1);
    } else {
      const int64_t m = (int64_t)gi * rsy + full - 1 - gj;  // mirror of gj; gj + 1's is before it
      if (two && full - 2 - gj != gj + 1) put(m - 1, true, e1 - o1, e0 - o0);
      else if (full - 1 - gj != gj) Y[m] = e0 - o0;
    }
  };
  if constexpr (SK > 1) {
    // Sum the waves' partial tiles in wave order; the operand chunks are dead
    // here (the K loop ends with a barrier).  Entry (i, j) of a partial tile is at
    // i TN + j.  The output's own operands are fetched first.
    T* red = sm.red;
    constexpr int PE = G::TM * G::TN / 2 / G::NT;  // pairs per thread
    pair ox[PE], op[PE];
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int e = tid + u * G::NT;
      operands(i0 + 2 * e / G::TN, j0 + 2 * e % G::TN, ox[u], op[u]);
    }
    auto sum = [&](const acc_t (&v)[BM][BN], pair (&out)[PE]) {
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; j += 2)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            *(pair*)(red + (sk * G::TM + (wm * BM + i) * 16 + Mma<T>::row(lk, r)) * G::TN + (wn * BN + j) * 16 +
                     2 * lr) = pair{v[i][j][r], v[i][j + 1][r]};
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PE; ++u) {
        const int e = tid + u * G::NT;
        pair v = ((const pair*)red)[e];
#pragma unroll
        for (int s = 1; s < SK; ++s) {
          const pair x = ((const pair*)red)[s * (G::TM * G::TN / 2) + e];
          v.x += x.x;
          v.y += x.y;
        }
        out[u] = v;
      }
      __syncthreads();  // the LDS is reused
    };
    pair v[PE], ev[PE];
    if constexpr (UNFOLD) sum(even, ev);
    sum(acc, v);
#pragma unroll
    for (int u = 0; u < PE; ++u) {
      const int e = tid + u * G::NT, gi = i0 + 2 * e / G::TN, gj = j0 + 2 * e % G::TN;
      if constexpr (UNFOLD) emit2(gi, gj, ev[u].x, ev[u].y, v[u].x, v[u].y);
      else emit(gi, gj, v[u].x, v[u].y, ox[u], op[u]);
    }
  } else if (MODE == MP_PLAIN && pairs && (uint64_t)(rs * ES) * G::TM >> 32 == 0 && i0 + G::TM <= M &&
             j0 + G::TN <= Nc && a.epi != EPI_DIV && !a.acc) {
    // a whole tile: uniform bases and one lane offset, the operands of 16 rows in
    // flight together
    const uint32_t vo = (wm * BM * 16 + Mma<T>::row(lk, 0)) * rsb + (wn * BN * 16 + 2 * lr) * ES;
    const int64_t o0 = i0 * rs + j0;
    constexpr int RS = Mma<T>::row(0, 1);  // rows between the outputs of a lane
#pragma unroll
    for (int i = 0; i < BM; ++i) {
      pair ox[4][BN / 2], op[4][BN / 2];
      if (a.epi == EPI_V) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < BN / 2; ++j) {
            const int64_t o = o0 + (i * 16 + r * RS) * rs + j * 32;
            ox[r][j] = *(const pair*)((const char*)(X + o) + vo);
            op[r][j] = Vp ? *(const pair*)((const char*)(Vp + o) + vo) : pair{0, 0};
          }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < BN / 2; ++j) {
          pair v{acc[i][2 * j][r], acc[i][2 * j + 1][r]};
          if (a.epi == EPI_V) {
            v.x += (op[r][j].x - shift) * ox[r][j].x;
            v.y += (op[r][j].y - shift) * ox[r][j].y;
          }
          *(pair*)((char*)(Y + o0 + (i * 16 + r * RS) * rs + j * 32) + vo) = v;
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pair ox[BN / 2], op[BN / 2];
        const int gi = i0 + (wm * BM + i) * 16 + Mma<T>::row(lk, r);
#pragma unroll
        for (int j = 0; j < BN / 2; ++j) operands(gi, j0 + (wn * BN + 2 * j) * 16 + 2 * lr, ox[j], op[j]);
#pragma unroll
        for (int j = 0; j < BN / 2; ++j) {
          const int gj = j0 + (wn * BN + 2 * j) * 16 + 2 * lr;
          if constexpr (UNFOLD)
            emit2(gi, gj, even[i][2 * j][r], even[i][2 * j + 1][r], acc[i][2 * j][r], acc[i][2 * j + 1][r]);
          else
            emit(gi, gj, acc[i][2 * j][r], acc[i][2 * j + 1][r], ox[j], op[j]);
        }
      }
  }
}

template <typename T, int BM, int BN, int WM, int WN, int SK, int MODE>
__device__ __forceinline__ void mp_tile(const ModeProd<T>& a, int64_t w,
                                        typename MpTile<T, BM, BN, WM, WN, SK>::Smem& sm) {
  // whole pieces: every row of every item starts on 16 bytes and is a multiple
  // of a piece long (folded columns: so is the row that they are the mirror in)
  constexpr int KU = MpVec<T>::KU;
  const bool whole = ((uintptr_t)a.X & 15) == 0 && a.rs % KU == 0 && a.ldx % KU == 0 &&
                     (MODE != MP_PLAIN || (a.Nc % KU == 0 && a.bstride % KU == 0)) &&
                     (MODE != MP_FOLD_R || a.full % KU == 0);
  if (MODE == MP_UNFOLD_L || MODE == MP_UNFOLD_R || whole)
    mp_tile_w<T, BM, BN, WM, WN, SK, MP_WHOLE, MODE>(a, w, sm);
  else
    mp_tile_w<T, BM, BN, WM, WN, SK, MP_ELEMENTS, MODE>(a, w, sm);
}

// The tile shapes of TileCfg: (BM, BN, WM, WN, SK).
#define TP3B_MP_32 2, 2, 1, 1, 4
#define TP3B_MP_32W8 2, 2, 1, 1, 8
#define TP3B_MP_64 2, 2, 2, 2, 1
#define TP3B_MP_64x128 2, 4, 2, 2, 1
#define TP3B_MP_128 4, 4, 2, 2, 1

}  // namespace tp3b
