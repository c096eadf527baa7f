// W_hat X (the dequantized weights of infer.hip's product) for few tokens:
// a decoding step, a small batch, or a narrow layer.
#include <type_traits>

#include "infer.h"

namespace ojbkq {
namespace {

// All lanes of the wave are past their LDS accesses (one wave's LDS operations
// execute in order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// 32 consecutive codes of a row from a feature that is a multiple of 32: BITS
// whole words, each code inside a window of two neighbouring ones.
template <int BITS>
struct Codes32 {
  typedef uint32_t Words __attribute__((ext_vector_type(BITS)));
  Words w;
  // whole: all 32 codes exist (words wi .. wi + BITS - 1 of the row do then)
  __device__ __forceinline__ void load(const uint32_t* row, int64_t wi, int64_t wpr, bool whole) {
    if (whole) {
      typedef uint32_t Any __attribute__((ext_vector_type(BITS), aligned(4)));
      const Any v = *reinterpret_cast<const Any*>(row + wi);
#pragma unroll
      for (int q = 0; q < BITS; ++q) w[q] = v[q];
    } else {
#pragma unroll
      for (int q = 0; q < BITS; ++q) w[q] = row[wi + q < wpr ? wi + q : wpr - 1];
    }
  }
  __device__ __forceinline__ float codef(int c) const {   // c a constant after unrolling
    const int b = c * BITS;
    if constexpr (BITS == 2 || BITS == 4 || BITS == 8) {
      // one shift and mask isolates a code in each byte, shared by the codes
      // at the same place of their bytes; byte-to-float converts take them out
      constexpr uint32_t kMask = BITS == 8 ? 0xffffffffu : BITS == 4 ? 0x0f0f0f0fu : 0x03030303u;
      const uint32_t y = (w[b >> 5] >> (b & 7)) & kMask;
      return (float)((y >> (b & 24)) & 0xffu);
    } else {
      constexpr uint32_t kMask = (1u << BITS) - 1u;
      const int lo = b >> 5, sh = b & 31;
      if (sh + BITS <= 32) return (float)((w[lo] >> sh) & kMask);
      return (float)(__builtin_amdgcn_alignbit(w[lo + 1 < BITS ? lo + 1 : lo], w[lo], sh) & kMask);
    }
  }
};

// Y = W_hat X for few tokens.  Such a product is bound by reading the codes
// (and for T near one by latency), so a workgroup takes few channels, 16 RB,
// for all features, and its eight waves split the features: chunks of 128 go
// round the waves, which meet only at the end, in LDS, where their sums are
// added in wave order.  Within a chunk lane l holds features 32 (l / 16) ..
// + 31 of channel l % 16, i.e. BITS whole words of a row, dequantized in
// registers straight into the A operand of four v_mfma_f32_16x16x32_f16
// (features 32 (l / 16) + 8 s .. + 7 in product s; the order of the features
// within a chunk is free as long as both operands agree).  The tokens, 16 NB
// of them per workgroup, are staged per wave in LDS in X's own [k][t] order
// and read by gfx950's transposing LDS read.  The next chunk's codes, scales
// and tokens are loaded while this one's products run.
// 4-bit codes, m = 4096: n = 4096, T = 1: 9 us (the code's bytes at the copy
// rate of 4.8 TB/s: 2 us; latency does the rest); n = 14336, T = 24: 24 us with
// the same codes again, 27 with those of forty layers in turn, from memory
// (7 us).  With W_hat formed first and 256 x 256 tiles: 162, 242 and 248 us.
template <int BITS, int RB, int NB>
__global__ __launch_bounds__(512) void dequant_few_kernel(DqArgs a) {
  constexpr int kChunk = 128, kTok = 16 * NB;
  // rows of kTok tokens; 64 halves of padding behind every 32 rows put the
  // four rows that the lane groups read at once in different banks
  constexpr int kWaveX = kChunk * kTok + 4 * 64;
  constexpr int kRed = RB * NB * 256;   // floats of a wave's sums
  constexpr int kLds = 8 * (kWaveX * 2 > kRed * 4 ? kWaveX * 2 : kRed * 4);
  __shared__ __align__(16) uint8_t lds[kLds];
  // A loop without masks for whole chunks, and loads without per-row checks,
  // where the registers hold a second copy of the code (us for n x 4096 x T
  // with / without the first: 14336 x 24, RB = NB = 2: 24.7 / 26.7; 4096 x
  // 512, RB = NB = 4, both: 300 / 71, with hundreds of registers spilled).
  constexpr bool kTwice = RB <= 2 && RB * NB <= 4;
  constexpr bool kQuick = RB * NB < 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;
  const int64_t J0 = (int64_t)blockIdx.x * (16 * RB), T0 = (int64_t)blockIdx.y * kTok;
  _Float16* const sX = reinterpret_cast<_Float16*>(lds) + wave * kWaveX;
  auto at = [&](int k, int t) { return k * kTok + (k >> 5) * 64 + t; };
  const int64_t nch = (a.m + kChunk - 1) / kChunk;
  const bool one_scale = a.g % 32 == 0 || a.g == a.m;   // of a lane's 32 features

  const uint32_t* prow[RB];
  const float *srow[RB], *zrow[RB];
#pragma unroll
  for (int x = 0; x < RB; ++x) {
    int64_t j = J0 + 16 * x + i16;
    j = j < a.n ? j : a.n - 1;   // feeds only rows that are not stored
    prow[x] = a.P + j * a.wpr;
    srow[x] = a.S + j * a.G;
    zrow[x] = a.Z + j * a.G;
  }

  struct Stage {
    Codes32<BITS> c[RB];
    float s[RB][2], z[RB][2];
    uint32_t x[16 * NB];   // tokens in flight
  };
  auto x_at = [&](int64_t k) { return a.X + x_row(a, k) * a.ldx; };
  // T >= 8: lane -> piece lane % (2 NB) of 8 tokens of row lane / (2 NB) +
  // 64 / (2 NB) q, one 16-byte load each at any alignment.  A piece that
  // reaches past the last token reads on into the next row, except in X's
  // last row, where its tokens are loaded singly.
  constexpr int kPieces = 2 * NB, kRowsPer = 64 / kPieces;
  const int piece = lane % kPieces, prow0 = lane / kPieces;
  const int64_t tp = T0 + 8 * piece;
  const bool by_piece = a.T >= 8;
  // e / T of an element number e < 14 * 64 as e * invT >> 16
  const int fewT = by_piece ? 1 : (int)a.T;
  const uint32_t invT = (65536u + fewT - 1) / fewT;
  typedef uint32_t Any4 __attribute__((ext_vector_type(4), aligned(2)));
  auto fetch = [&](int64_t c, Stage& st) {
    const int64_t k0 = c * kChunk, kc = k0 + 32 * g4;
    const bool whole = k0 + kChunk <= a.m;
#pragma unroll
    for (int x = 0; x < RB; ++x) {
      st.c[x].load(prow[x], (kc >> 5) * BITS, a.wpr, whole);
      const uint32_t g0 = (uint32_t)(kc < a.m ? kc : a.m - 1) / (uint32_t)a.g;
      st.s[x][0] = srow[x][g0];
      st.z[x][0] = zrow[x][g0];
      if (one_scale) {
        st.s[x][1] = st.s[x][0];
        st.z[x][1] = st.z[x][0];
      } else {
        const uint32_t g1 = (uint32_t)(kc + 16 < a.m ? kc + 16 : a.m - 1) / (uint32_t)a.g;
        st.s[x][1] = srow[x][g1];
        st.z[x][1] = zrow[x][g1];
      }
    }
    if (kQuick && by_piece && !a.perm && k0 + kChunk < a.m) {
      // (whole, and without X's last row)
      const uint16_t* src = a.X + (k0 + prow0) * a.ldx + (tp < a.T ? tp : 0);
#pragma unroll
      for (int q = 0; q < kChunk / kRowsPer; ++q) {
        const Any4 v = *reinterpret_cast<const Any4*>(src);
        src += kRowsPer * a.ldx;
#pragma unroll
        for (int e = 0; e < 4; ++e) st.x[4 * q + e] = v[e];
      }
    } else if (by_piece) {
#pragma unroll
      for (int q = 0; q < kChunk / kRowsPer; ++q) {
        const int64_t k = k0 + prow0 + kRowsPer * q;
        Any4 v = Any4{0u, 0u, 0u, 0u};
        if (k < a.m && tp < a.T) {
          const int64_t r = x_row(a, k);
          const uint16_t* src = a.X + r * a.ldx + tp;
          if (x_piece_inside(r, tp, a.m, a.T)) {
            v = *reinterpret_cast<const Any4*>(src);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (tp + e < a.T) v[e / 2] |= (uint32_t)src[e] << (16 * (e & 1));
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) st.x[4 * q + e] = v[e];
      }
    } else if constexpr (NB == 1) {
      // up to seven tokens: element e = lane + 64 q is token e % T of row e / T
#pragma unroll
      for (int q = 0; q < 14; ++q) {
        if (q >= 2 * fewT) break;
        const uint32_t e = lane + 64 * q, k = e * invT >> 16, t = e - k * fewT;
        st.x[q] = k0 + k < a.m ? x_at(k0 + k)[t] : 0u;
      }
    }
  };
  // tokens of the stage to LDS (a wave's own area: no workgroup barrier)
  auto put = [&](const Stage& st) {
    wave_sync();   // the previous chunk's reads
    if (by_piece) {
#pragma unroll
      for (int q = 0; q < kChunk / kRowsPer; ++q)
        *reinterpret_cast<uint4*>(sX + at(prow0 + kRowsPer * q, 8 * piece)) =
            make_uint4(st.x[4 * q], st.x[4 * q + 1], st.x[4 * q + 2], st.x[4 * q + 3]);
    } else if constexpr (NB == 1) {
#pragma unroll
      for (int q = 0; q < 14; ++q) {
        if (q >= 2 * fewT) break;
        const uint32_t e = lane + 64 * q, k = e * invT >> 16, t = e - k * fewT;
        sX[at(k, t)] = __builtin_bit_cast(_Float16, (uint16_t)st.x[q]);
      }
    }
    wave_sync();
  };

  f4 acc[RB][NB];
#pragma unroll
  for (int x = 0; x < RB; ++x)
#pragma unroll
    for (int y = 0; y < NB; ++y) acc[x][y] = f4{0.f, 0.f, 0.f, 0.f};
  auto products = [&](int64_t c, const Stage& st, auto whole) {
    // codes of this lane that exist (all but in a last ragged chunk; one past
    // the end need not give a finite weight)
    const int64_t left = a.m - (c * kChunk + 32 * g4);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      h8 fb[NB];
#pragma unroll
      for (int y = 0; y < NB; ++y) {
        auto tr = [&](int k) {
          const _Float16* p = sX + at(k + (i16 >> 2), 16 * y + 4 * (i16 & 3));
          return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (s4 __attribute__((address_space(3)))*)(const_cast<_Float16*>(p)));
        };
        const s4 lo = tr(32 * g4 + 8 * s), hi = tr(32 * g4 + 8 * s + 4);
        fb[y] = __builtin_bit_cast(h8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int x = 0; x < RB; ++x) {
        const float sc = st.s[x][s >> 1], zc = st.z[x][s >> 1];
        h8 fa;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          // two roundings, as everywhere: the asm keeps the float32 products
          float p0 = sc * (st.c[x].codef(8 * s + e) - zc);
          float p1 = sc * (st.c[x].codef(8 * s + e + 1) - zc);
          __asm__("" : "+v"(p0), "+v"(p1));
          if (!whole) {
            p0 = 8 * s + e < left ? p0 : 0.f;
            p1 = 8 * s + e + 1 < left ? p1 : 0.f;
          }
          const h2 w2 = to_f16x2(p0, p1);
          fa[e] = w2.x;
          fa[e + 1] = w2.y;
        }
#pragma unroll
        for (int y = 0; y < NB; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, fb[y], acc[x][y], 0, 0, 0);
      }
    }
  };

  Stage st;
  if (wave < nch) {
    fetch(wave, st);
    for (int64_t c = wave; c < nch; c += 8) {
      put(st);
      const Stage cur = st;
      if (c + 8 < nch) fetch(c + 8, st);
      const bool whole = (c + 1) * kChunk <= a.m;
      if constexpr (!kTwice)
        products(c, cur, whole);
      else if (whole)
        products(c, cur, std::true_type{});
      else
        products(c, cur, std::false_type{});
    }
  }

  // the waves' sums, in wave order: lane l holds D[4 (l / 16) + r][l % 16]
  __syncthreads();
  float* const red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int x = 0; x < RB; ++x)
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[wave * kRed + (16 * x + 4 * g4 + r) * kTok + 16 * y + i16] = acc[x][y][r];
  __syncthreads();
  for (int e = tid; e < kRed; e += 512) {
    float v = red[e];
#pragma unroll
    for (int w = 1; w < 8; ++w) v += red[w * kRed + e];
    const int64_t j = J0 + e / kTok, t = T0 + e % kTok;
    if (j < a.n && t < a.T) a.Y[j * a.ldy + t] = v;
  }
}

template <int BITS, int NB>
hipError_t launch_few_rb(const DqArgs& a, hipStream_t s) {
  // as many channels per workgroup as leave one for every CU: the tokens are
  // read once per workgroup
  const int64_t gy = (a.T + 16 * NB - 1) / (16 * NB);
  auto grid = [&](int rb) { return dim3((unsigned)((a.n + 16 * rb - 1) / (16 * rb)), (unsigned)gy); };
  if ((a.n + 63) / 64 * gy >= 256)
    dequant_few_kernel<BITS, 4, NB><<<grid(4), dim3(512), 0, s>>>(a);
  else if ((a.n + 31) / 32 * gy >= 256)
    dequant_few_kernel<BITS, 2, NB><<<grid(2), dim3(512), 0, s>>>(a);
  else
    dequant_few_kernel<BITS, 1, NB><<<grid(1), dim3(512), 0, s>>>(a);
  return hipGetLastError();
}

template <int BITS>
hipError_t launch_few(const DqArgs& a, hipStream_t s) {
  if (a.T <= 16) return launch_few_rb<BITS, 1>(a, s);
  if (a.T <= 32) return launch_few_rb<BITS, 2>(a, s);
  return launch_few_rb<BITS, 4>(a, s);
}

}  // namespace

hipError_t launch_dequant_few(const DqArgs& a, int bits, hipStream_t stream) {
  switch (bits) {
    case 1: return launch_few<1>(a, stream);
    case 2: return launch_few<2>(a, stream);
    case 3: return launch_few<3>(a, stream);
    case 4: return launch_few<4>(a, stream);
    case 5: return launch_few<5>(a, stream);
    case 6: return launch_few<6>(a, stream);
    case 7: return launch_few<7>(a, stream);
    case 8: return launch_few<8>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ojbkq
