// laim_wide.hip -- the round machine on codes whose state exceeds what the
// resident form holds: one persistent block of 1024 threads per shot, the
// messages in LDS and, past its end, in a block-private stretch of device
// memory that the caches hold.
//
// A sweep is the two phases as written, in place: word (c, j) holds m_{c->v}
// after a check phase and m_{v->c} after a qubit phase. In the qubit phase the
// owner of a qubit reads its d_v messages, forms the d_v sums (BP-LLR1, in
// ascending check order) and writes them to the same words; in the check phase
// the owner of a check does the same with its d_c words (BP-LLR2). No word has
// two users in a phase, so there is no second buffer, and nothing about the
// messages stays in registers: the size of a code is bounded by its words.
//
// What bounds it: the LDS, where a message is read twice and written twice a
// sweep, and the reads of the messages past it; a block alone on its CU also
// waits for their latency, so the tiles of a wavefront are worked on several
// at a time. Measured, 256 shots in flight, min-sum: 3.0 us a sweep on 3D
// membrane L = 12 (5,184 checks, all in LDS; 1.6 us at the LDS's own rates),
// 7.5 us on L = 16 (12,288 checks, 22% of the words past the LDS), 7.3 us on
// the point sector at L = 19, 28 us at L = 24 (54% past it). The stream form
// moves every message through HBM each sweep, 34 us for 256 shots of membrane
// L = 16 at 6 TB/s, and takes a launch per sweep and phase. A decode of 1,024
// shots at p = 0.03, 64 rounds: 43.5 ms in the stream form, 11.3 ms here, of
// which 9 ms are the six shots that never clear. This form was the faster one
// at every size tried, 32 to 4,096 shots of membrane L = 13, 16, point L = 22, 24
// and 2D toric L = 100, with both rules (1.1 to 20 times).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device_math.h"
#include "laim_internal.h"

namespace laim {

namespace {

constexpr int kWideThreads = 1024;
constexpr int kWideWaves = kWideThreads / 64;
constexpr int kWideMaxChecks = 32 * kWideThreads;   // a thread's syndrome bits are one word
constexpr int kWideMaxQubits = 64 * kWideThreads;   // and its wavefront's qubit tiles one 64-bit mask
constexpr int kWideDummy = 4;  // first words of the LDS: the messages of the qubits that pad the last tile
constexpr int kWideCtrl = 16;
// control words
constexpr int kWcQueue = 0, kWcInit = 1, kWcFlips = 2, kWcLive = 3, kWcAct0 = 4, kWcAct1 = 5, kWcChg = 6;

struct WideArgs {
  const uint8_t* e0;  // [nshots][n] initial errors, or null when s0 is given
  const uint8_t* s0;  // [nshots][m] start syndromes, or null: H e0
  int32_t r0;         // number of the first round (the clocks' Philox counter)
  uint64_t shot0;
  int32_t nshots;
  uint32_t* counter;      // queue head, or null: block b runs shot b only
  const uint32_t* table;  // [n padded to 64][wide_row(DV)] byte offsets of each qubit's messages,
                          // ascending check
  int32_t ltiles;         // tiles of 64 checks whose messages are in LDS; the others follow in `over`
  float* over;            // [blocks][over_words]
  int64_t over_words;
  float* copy;            // [blocks][copy_words]: the messages before a compared sweep
  int64_t copy_words;
  uint8_t* z;
  uint8_t* s;
  int32_t* tclr;
  float* L;
};

template <int I>
struct IntTag {
  static constexpr int value = I;
};

// Entries per qubit in the table: one vector load.
constexpr int wide_row(int dv) { return dv == 3 ? 4 : dv; }

// The byte offset of each qubit's messages, and the queue head cleared.
__global__ void __launch_bounds__(256) wide_setup(DevCode c, int32_t row, uint32_t* __restrict__ table,
                                                  uint32_t* counter) {
  const int32_t i = (int32_t)(bid_x() * bdim_x() + tid_x());
  if (i == 0) counter[0] = 0u;
  if (i >= (c.n + 63) / 64 * 64 * row) return;
  const int32_t v = i / row, q = i - v * row;
  int32_t w = q;  // a padding qubit: the dummy words
  if (v < c.n && q < c.dvmax) {
    const int32_t e = c.var_edge[(int64_t)v * c.dvmax + q];  // regular codes: every entry is an edge
    w = kWideDummy + resident_msg_word(c.dcmax, edge_check(e), edge_slot(e));
  }
  table[i] = 4u * (uint32_t)w;
}

// The check rule (BP-LLR2) of a regular check from its inputs x. Min-sum runs
// with alpha <= 1 (its outputs cannot reach the clamp).
template <int DC, int BP>
__device__ __forceinline__ void wide_check_rule(const KParams& kp, const float* x, uint32_t sigma_neg, float* out) {
  if constexpr (BP == 0) {
    uint32_t par = sigma_neg << 31;
#pragma unroll
    for (int j = 0; j + 1 < DC; j += 2) par = xor3(par, __float_as_uint(x[j]), __float_as_uint(x[j + 1]));
    const float alpha_s = __uint_as_float(__float_as_uint(kp.alpha) ^ (par & 0x80000000u));
    float ex[DC];  // smallest |m| over the other inputs
    min_others<DC>(x, ex);
#pragma unroll
    for (int j = 0; j < DC; ++j) {
      const float v = alpha_s * ex[j];
      out[j] = __uint_as_float(__float_as_uint(v) ^ (__float_as_uint(x[j]) & 0x80000000u));
    }
  } else {
    float acc[DC];
    boxplus_others<DC, true>(x, DC, acc);
#pragma unroll
    for (int j = 0; j < DC; ++j) out[j] = __builtin_amdgcn_fmed3f(sigma_neg ? -acc[j] : acc[j], -kp.clamp, kp.clamp);
  }
}

template <int DC, int DV, int BP>
__global__ void __launch_bounds__(kWideThreads) wide_kernel(DevCode c, KParams kp, WideArgs a) {
  extern __shared__ __align__(16) float lds[];
  constexpr int T = kWideThreads, NW = kWideWaves, R = wide_row(DV);
  constexpr int TW = DC * kResSlotStride;  // words of a tile of 64 checks
  const int32_t t = tid_x();
  const int32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int32_t tiles = (c.m + 63) >> 6, qtiles = (c.n + 63) >> 6;
  const int32_t wl = kWideDummy + a.ltiles * TW;     // words in LDS
  const int32_t words = kWideDummy + tiles * TW;     // and in all
  const int32_t nw = (c.n + 31) >> 5, mw = (c.m + 31) >> 5;
  uint32_t* flw = reinterpret_cast<uint32_t*>(lds + wl);  // [nw] flip requests
  uint32_t* zw = flw + nw;                                // [nw] correction
  uint32_t* sw = zw + nw;                                 // [mw] syndrome
  int32_t* ctrl = reinterpret_cast<int32_t*>(sw + mw);
  float* over = a.over + (int64_t)bid_x() * a.over_words;  // word w >= wl is over[w - wl]
  float* copy = a.copy + (int64_t)bid_x() * a.copy_words;
  const float C = kp.clamp, pi = kp.pi;
  const int32_t cpt = (c.m + T - 1) / T;  // checks t + k T of this thread, k < cpt <= 32
  const float thr = c.thr[DC];
  // a message by its byte offset
  const uint32_t lbytes = 4u * (uint32_t)wl;
  char* const lb = reinterpret_cast<char*>(lds);
  char* const ob = reinterpret_cast<char*>(over);
  auto ld = [&](uint32_t o) -> float {
    return o < lbytes ? *reinterpret_cast<const float*>(lb + o) : *reinterpret_cast<const float*>(ob + (o - lbytes));
  };

  // Wavefront w owns the qubit tiles and the check tiles w, w + 16, ... The
  // offsets of its k-th qubit tile; bit k of far[q]: the q-th message of a
  // qubit of that tile lies past the LDS.
  const int32_t nq = (qtiles - wave + NW - 1) / NW;  // this wavefront's qubit tiles (may be 0)
  const int32_t nc = (tiles - wave + NW - 1) / NW;   // its check tiles,
  const int32_t nl = min(nc, max(0, (a.ltiles - wave + NW - 1) / NW));  // the first nl of them in LDS
  auto fetch = [&](int32_t k, uint32_t* o) {
    const uint32_t at = (uint32_t)(k * T + t) * (R * 4u);
    __builtin_memcpy(o, __builtin_assume_aligned(reinterpret_cast<const char*>(a.table) + at, R * 4), R * 4);
  };
  uint64_t far[DV], far_any = 0ull;
#pragma unroll
  for (int q = 0; q < DV; ++q) far[q] = 0ull;
  for (int32_t k = 0; k < nq; ++k) {
    uint32_t o[R];
    fetch(k, o);
#pragma unroll
    for (int q = 0; q < DV; ++q)
      if (__builtin_amdgcn_ballot_w64(o[q] >= lbytes) != 0ull) far[q] |= 1ull << k;
  }
#pragma unroll
  for (int q = 0; q < DV; ++q) far_any |= far[q];

  // BP-LLR1 in place for U of the wavefront's qubit tiles from the k-th on,
  // all their messages in LDS: the reads are in flight together.
  auto sum_others = [&](const float* mm, int q) {
    float acc = pi;
#pragma unroll
    for (int p = 0; p < DV; ++p)
      if (p != q) acc = acc + mm[p];
    return __builtin_amdgcn_fmed3f(acc, -C, C);
  };
  auto qubits = [&](auto ucount, int32_t k) {
    constexpr int U = decltype(ucount)::value;
    uint32_t o[U][R];
    float mm[U][DV];
#pragma unroll
    for (int u = 0; u < U; ++u) fetch(k + u, o[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < DV; ++q) mm[u][q] = *reinterpret_cast<const float*>(lb + o[u][q]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < DV; ++q) *reinterpret_cast<float*>(lb + o[u][q]) = sum_others(mm[u], q);
  };
  // The same where some messages lie past the LDS. Lanes on the other side of
  // the line read and write a scratch word there (word 0 of the LDS, the last
  // of `over`), so that both sides' accesses need no branch per lane.
  auto far_qubits = [&](auto ucount, int32_t k) {
    constexpr int U = decltype(ucount)::value;
    uint32_t o[U][R];
    float mm[U][DV], g[U][DV];
#pragma unroll
    for (int u = 0; u < U; ++u) fetch(k + u, o[u]);
    const uint32_t oscr = (uint32_t)(a.over_words - 64 + lane) * 4u;
    constexpr uint64_t mask = (1ull << U) - 1ull;
#pragma unroll
    for (int q = 0; q < DV; ++q)
      if ((far[q] >> k) & mask) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          g[u][q] = *reinterpret_cast<const float*>(ob + (o[u][q] < lbytes ? oscr : o[u][q] - lbytes));
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) g[u][q] = 0.0f;
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < DV; ++q) {
        const float m = *reinterpret_cast<const float*>(lb + (o[u][q] < lbytes ? o[u][q] : 0u));
        mm[u][q] = o[u][q] < lbytes ? m : g[u][q];
      }
#pragma unroll
    for (int q = 0; q < DV; ++q) {
      float x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u] = sum_others(mm[u], q);
        *reinterpret_cast<float*>(lb + (o[u][q] < lbytes ? o[u][q] : 0u)) = x[u];
      }
      if ((far[q] >> k) & mask) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          *reinterpret_cast<float*>(ob + (o[u][q] < lbytes ? oscr : o[u][q] - lbytes)) = x[u];
      }
    }
  };
  auto qubit_phase = [&]() {
    constexpr int U = DV >= 3 ? 4 : 8, UF = DV >= 3 ? 3 : 4;
    int32_t k = 0;
    while (k < nq) {
      const uint64_t f = far_any >> k;
      if (k + U <= nq && !(f & ((1ull << U) - 1ull))) {
        qubits(IntTag<U>(), k);
        k += U;
      } else if (k + 2 <= nq && !(f & 3ull)) {
        qubits(IntTag<2>(), k);
        k += 2;
      } else if (!(f & 1ull)) {
        qubits(IntTag<1>(), k);
        ++k;
      } else if (k + UF <= nq) {
        far_qubits(IntTag<UF>(), k);
        k += UF;
      } else {
        far_qubits(IntTag<1>(), k);
        ++k;
      }
    }
  };

  // BP-LLR2 in place for U of the wavefront's check tiles from the k-th on,
  // all in LDS or all past it. The checks that pad the last tile are updated
  // like the others (nothing reads them); `diff` leaves them out.
  uint32_t sb = 0u;  // bit k: syndrome of check t + k T
  uint32_t diff = 0u;
  auto checks = [&](auto ucount, float* base, int32_t k, bool cmp, bool keep) {
    constexpr int U = decltype(ucount)::value;
    float x[U][DC];
    const int32_t w0 = kWideDummy + (wave + NW * k) * TW + lane;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < DC; ++j) x[u][j] = base[w0 + u * NW * TW + j * kResSlotStride];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float out[DC];
      wide_check_rule<DC, BP>(kp, x[u], ((sb >> (k + u)) ^ (uint32_t)DC) & 1u, out);
#pragma unroll
      for (int j = 0; j < DC; ++j) base[w0 + u * NW * TW + j * kResSlotStride] = out[j];
      float* const cw = copy + (w0 + u * NW * TW);
      if (cmp) {
        uint32_t dk = 0u;
#pragma unroll
        for (int j = 0; j < DC; ++j) dk |= __float_as_uint(cw[j * kResSlotStride]) ^ __float_as_uint(out[j]);
        diff |= t + (k + u) * T < c.m ? dk : 0u;
      }
      if (keep) {
#pragma unroll
        for (int j = 0; j < DC; ++j) cw[j * kResSlotStride] = out[j];
      }
    }
  };
  auto check_phase = [&](bool cmp, bool keep) {
    constexpr int U = BP == 0 ? 4 : 1;
    int32_t k = 0;
    for (; k + U <= nl; k += U) checks(IntTag<U>(), lds, k, cmp, keep);
    for (; k < nl; ++k) checks(IntTag<1>(), lds, k, cmp, keep);
    float* const past = over - wl;  // word w >= wl
    for (; k + U <= nc; k += U) checks(IntTag<U>(), past, k, cmp, keep);
    for (; k < nc; ++k) checks(IntTag<1>(), past, k, cmp, keep);
  };

  for (int32_t turn = 0;; ++turn) {
    int32_t idx = (int32_t)bid_x();
    if (a.counter) {
      __syncthreads();
      if (t == 0) ctrl[kWcQueue] = (int32_t)atomicAdd(a.counter, 1u);
      __syncthreads();
      idx = ctrl[kWcQueue];
    } else if (turn) {
      break;
    }
    if (idx >= a.nshots) break;
    const uint64_t shot = a.shot0 + (uint64_t)idx;

    // ---- start: every message 0 (read as m_{v->c} by the shot's first check
    // phase), z = 0, s = H e0 (accumulated from the error's qubits) or s0
    for (int32_t w = t; w < wl; w += T) lds[w] = 0.0f;
    for (int32_t w = t; w < words - wl; w += T) over[w] = 0.0f;
    for (int32_t w = t; w < 2 * nw + mw; w += T) flw[w] = 0u;
    if (t < kWideCtrl && t != kWcQueue) ctrl[t] = 0;
    __syncthreads();
    sb = 0u;
    if (a.s0) {
      const uint8_t* row0 = a.s0 + (int64_t)idx * c.m;
      for (int32_t k = 0; k < cpt; ++k) {
        const int32_t ch = t + k * T;
        if (ch < c.m && (row0[ch] & 1u)) {
          sb |= 1u << k;
          atomicOr(&sw[ch >> 5], 1u << (ch & 31));
        }
      }
    } else {
      const uint8_t* row0 = a.e0 + (int64_t)idx * c.n;
#pragma unroll 4
      for (int32_t v = t; v < c.n; v += T) {
        if (!(row0[v] & 1u)) continue;
#pragma unroll
        for (int q = 0; q < DV; ++q) {
          const int32_t c2 = edge_check(c.var_edge[(int64_t)v * DV + q]);
          atomicXor(&sw[c2 >> 5], 1u << (c2 & 31));
        }
      }
      __syncthreads();
      for (int32_t k = 0; k < cpt; ++k) {
        const int32_t ch = t + k * T;
        if (ch < c.m) sb |= ((sw[ch >> 5] >> (ch & 31)) & 1u) << k;
      }
    }
    if (sb) ctrl[kWcInit] = 1;
    __syncthreads();
    int32_t tclr = ctrl[kWcInit] ? -1 : 0;
    bool working = !(kp.retire && tclr >= 0);
    bool fresh = true;  // no sweep yet
    bool conv = false;  // the messages are a fixed point of the sweep for the current syndrome
    uint32_t noev = 0u;  // active checks that failed Evidence at this fixed point

    // (one shot per block: every condition on the round's state is uniform)
    for (int32_t rr = 0; rr < kp.rounds && working; ++rr) {
      const int32_t r = a.r0 + rr;
      __syncthreads();
      if (t == 0) {
        ctrl[((rr + 1) & 1) ? kWcAct1 : kWcAct0] = 0;
        ctrl[kWcFlips] = 0;
        ctrl[kWcLive] = 0;
        ctrl[kWcChg] = 0;
      }
      __syncthreads();
      const bool same_state = conv;
      if (!conv) {
        for (int32_t it = 0; it < kp.iters; ++it) {
          // With the exact shortcuts the last sweep of a round compares each
          // new message with the one it replaces, which the sweep before it
          // kept in `copy`: a sweep that changes nothing is repeated exactly
          // by every later one until a flip. A shot's first sweep (from
          // m_{v->c} = 0) is another map and never counts.
          const bool cmp = kp.skip && it == kp.iters - 1 && !fresh;
          const bool keep = kp.skip && it == (kp.iters > 1 ? kp.iters - 2 : 0);
          if (!fresh) {
            qubit_phase();
            __syncthreads();
          }
          diff = 0u;
          check_phase(cmp, keep);
          fresh = false;
          if (cmp && diff) ctrl[kWcChg] = 1;
          __syncthreads();
          if (cmp && ctrl[kWcChg] == 0) conv = true;
        }
      }

      // ---- feedback, as in the resident form: every active check whose
      // beliefs pass Evidence and whose clock rang requests its move
      if (!same_state) noev = 0u;
      uint32_t act = sb & ~noev;
      int32_t nflip = 0;
#pragma unroll 1
      while (act) {
        const int32_t k = __builtin_ctz(act);
        act &= act - 1u;
        const int32_t ch = t + k * T;
        const int32_t* nb = c.chk_var + (int64_t)ch * DC;
        int32_t nbv[DC];
#pragma unroll
        for (int j = 0; j < DC; ++j) nbv[j] = nb[j];
        float Lv[DC];
        float Lmax = -__builtin_inff();
#pragma unroll
        for (int j = 0; j < DC; ++j) {
          float acc = pi;
#pragma unroll
          for (int q = 0; q < DV; ++q) acc = acc + ld(a.table[(int64_t)nbv[j] * R + q]);
          acc = clampf(acc, C);
          Lv[j] = acc;
          if (j == 0 || acc > Lmax) Lmax = acc;
        }
        if (kp.evidence && !(Lmax >= thr)) {
          noev |= 1u << k;
          continue;
        }
        const Philox4 w = philox4x32_10((uint32_t)shot, (uint32_t)(shot >> 32), (uint32_t)ch, ((uint32_t)r << 4) | 1u,
                                        (uint32_t)kp.seed, (uint32_t)(kp.seed >> 32));
        if (!below(w.w0, kp.mask_bound)) continue;
        uint32_t ntie = 0;
#pragma unroll
        for (int j = 0; j < DC; ++j) ntie += (Lv[j] == Lmax) ? 1u : 0u;
        uint32_t pick = (uint32_t)(((uint64_t)w.w1 * (uint64_t)ntie) >> 32);
        uint32_t fmask = 0u, pos = 0u;
#pragma unroll
        for (int j = 0; j < DC; ++j) {
          if (Lv[j] > 0.0f) pos |= 1u << j;
          if (Lv[j] == Lmax && !fmask) {
            if (pick == 0)
              fmask = 1u << j;
            else
              --pick;
          }
        }
        if (!fmask) continue;
        if (kp.move && pos) fmask = pos;
#pragma unroll 1
        while (fmask) {
          const int32_t jj = __builtin_ctz(fmask);
          fmask &= fmask - 1u;
          const int32_t v = nb[jj];
          const uint32_t bit = 1u << (v & 31);
          uint32_t had = 0u;
          if (kp.conflict == kConflictOr) {
            if (atomicOr(&flw[v >> 5], bit) & bit) continue;  // already requested
          } else {
            had = atomicXor(&flw[v >> 5], bit) & bit;
          }
          atomicXor(&zw[v >> 5], bit);
#pragma unroll
          for (int q = 0; q < DV; ++q) {
            const int32_t c2 = edge_check(c.var_edge[(int64_t)v * DV + q]);
            atomicXor(&sw[c2 >> 5], 1u << (c2 & 31));
          }
          nflip += had ? -1 : 1;
        }
      }
      if (nflip) atomicAdd(&ctrl[kWcFlips], nflip);
      if (sb & ~noev) ctrl[kWcLive] = 1;  // an active check passed the Evidence test
      __syncthreads();
      const int32_t nfl = ctrl[kWcFlips];
      if (nfl) {
        sb = 0u;
        for (int32_t k = 0; k < cpt; ++k) {
          const int32_t ch = t + k * T;
          if (ch < c.m) sb |= ((sw[ch >> 5] >> (ch & 31)) & 1u) << k;
        }
        for (int32_t w = t; w < nw; w += T) flw[w] = 0u;
      }
      int32_t* any = &ctrl[(rr & 1) ? kWcAct1 : kWcAct0];
      if (sb) *any = 1;
      __syncthreads();
      if (!*any && tclr < 0) tclr = r + 1;
      if (nfl) conv = false;  // the syndrome changed
      if (kp.retire && tclr >= 0) working = false;
      // frozen: nothing flipped at a fixed point and no active check passes
      // Evidence, so every later round repeats this one
      if (conv && !ctrl[kWcLive]) working = false;
    }

    // ---- results
    uint8_t* zrow = a.z + (int64_t)idx * c.n;
    for (int32_t v = t; v < c.n; v += T) zrow[v] = (uint8_t)((zw[v >> 5] >> (v & 31)) & 1u);
    uint8_t* srow = a.s + (int64_t)idx * c.m;
    for (int32_t k = 0; k < cpt; ++k)
      if (t + k * T < c.m) srow[t + k * T] = (uint8_t)((sb >> k) & 1u);
    if (t == 0) a.tclr[idx] = tclr;
    if (a.L) {
      for (int32_t v = t; v < c.n; v += T) {
        float acc = pi;
#pragma unroll
        for (int q = 0; q < DV; ++q) acc = acc + ld(a.table[(int64_t)v * R + q]);
        a.L[(int64_t)idx * c.n + v] = clampf(acc, C);
      }
    }
    __syncthreads();  // the results are read from LDS before the next shot clears it
  }
}

typedef void (*WideKernel)(DevCode, KParams, WideArgs);
struct WideVariant {
  int dc, dv, bp;
  WideKernel fn;
};
#define LAIM_WIDE(DC, DV) {DC, DV, 0, wide_kernel<DC, DV, 0>}, {DC, DV, 1, wide_kernel<DC, DV, 1>}
const WideVariant kWideVariants[] = {LAIM_WIDE(4, 2), LAIM_WIDE(6, 2), LAIM_WIDE(4, 4), LAIM_WIDE(6, 3)};

const WideVariant* wide_variant(const DevCode& c, int bp) {
  for (const auto& v : kWideVariants)
    if (v.dc == c.dcmax && v.dv == c.dvmax && v.bp == bp) return &v;
  return nullptr;
}

size_t al256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

// Min-sum with alpha > 1 (whose outputs need a clamp), the sequential rule and
// irregular codes keep the stream form; so do codes of at most 4,096 checks,
// which run resident but for those cases and would leave threads of a block
// without a check.
// Codes of qubit degree 2 or 3 with more than half of their messages past the
// LDS (which holds about 38,000) run faster in the stream form once there are
// more shots than half of one of its tiles. Measured, ms in the stream form and
// here, 1,024 shots, min-sum, 4 rounds: 2D toric L = 150, 90,000 messages, 11.9 /
// 11.8; L = 160, 102,400, 13.4 / 14.9; L = 180, 129,600, 17.1 / 21.8; 3D point L = 24,
// 82,944, 11.1 / 9.3; L = 26, 105,456, 14.0 / 15.6; bicycle codes, 98,304 15.7 / 13.2 and
// 153,600 24.4 / 27.7. Sum-product, L = 150 16.5 / 16.3, L = 176 22.8 / 23.9. Up to 128
// shots this form was the faster one at every size, and membrane codes (qubit degree 4)
// at every number of shots up to L = 22, 127,776 messages, 21.7 / 17.6.
static bool wide_pays(const DevCode& c, int32_t nshots) {
  const int64_t most = c.dvmax == 2 ? 92000 : c.dvmax == 3 ? 110000 : INT64_MAX;
  return nshots <= 128 || (int64_t)c.m * c.dcmax <= most;
}

bool wide_ok(const DevCode& c, const KParams& kp, int32_t nshots) {
  return c.regular && c.m > kWideMinChecks && c.m <= kWideMaxChecks && c.n <= kWideMaxQubits &&
         kp.conflict != kConflictSequential && !(kp.bp == 0 && kp.alpha > 1.0f) && wide_pays(c, nshots) &&
         wide_variant(c, kp.bp) != nullptr;
}

hipError_t launch_wide(const DevCode& c, const KParams& kp, const uint8_t* e0, uint64_t shot0, int32_t nshots,
                       void* ws, size_t ws_bytes, uint8_t* z, uint8_t* s, int32_t* tclr, float* L, hipStream_t st,
                       const uint8_t* s0, int32_t r0) {
  if (nshots <= 0) return hipSuccess;
  const WideVariant* var = wide_variant(c, kp.bp);
  if (!var) return hipErrorInvalidValue;
  int dev = 0, lds_max = 0, cus = 0;
  (void)hipGetDevice(&dev);
  if (hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || lds_max <= 0)
    lds_max = 64 * 1024;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
  const int32_t tiles = (c.m + 63) / 64;
  const int64_t tile_bytes = (int64_t)c.dcmax * kResSlotStride * 4;
  const int64_t fixed = (int64_t)(kWideDummy + 2 * ((c.n + 31) / 32) + (c.m + 31) / 32 + kWideCtrl) * 4;
  const int64_t fit = (lds_max - fixed) / tile_bytes;
  if (fit < 0) return hipErrorInvalidConfiguration;
  WideArgs a;
  a.ltiles = (int32_t)std::min<int64_t>(tiles, fit);
  const int64_t words = (int64_t)tiles * c.dcmax * kResSlotStride;
  a.over_words = (words - (int64_t)a.ltiles * c.dcmax * kResSlotStride + 63) / 64 * 64 + 64;  // and 64 scratch words
  a.copy_words = kp.skip ? (kWideDummy + words + 63) / 64 * 64 : 0;
  // workspace: queue head, table, then the blocks' messages and copies
  const int32_t rowlen = wide_row(c.dvmax);
  const size_t entries = (size_t)((c.n + 63) / 64 * 64) * rowlen;
  const size_t head = 256 + al256(entries * 4);
  const size_t per_block = (size_t)(a.over_words + a.copy_words) * 4;
  int64_t blocks = std::min<int64_t>(nshots, cus);
  if (per_block) {
    if (ws_bytes < head + per_block) return hipErrorInvalidValue;
    blocks = std::min<int64_t>(blocks, (int64_t)((ws_bytes - head) / per_block));
  }
  char* p = static_cast<char*>(ws);
  uint32_t* counter = reinterpret_cast<uint32_t*>(p);
  uint32_t* table = reinterpret_cast<uint32_t*>(p + 256);
  a.table = table;
  a.over = reinterpret_cast<float*>(p + head);
  a.copy = a.over + blocks * a.over_words;
  a.e0 = e0;
  a.s0 = s0;
  a.r0 = r0;
  a.shot0 = shot0;
  a.nshots = nshots;
  a.counter = blocks < nshots ? counter : nullptr;
  a.z = z;
  a.s = s;
  a.tclr = tclr;
  a.L = L;
  hipLaunchKernelGGL(wide_setup, dim3((unsigned)((entries + 255) / 256)), dim3(256), 0, st, c, rowlen, table, counter);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const WideKernel fn = var->fn;
  const size_t lds_bytes = (size_t)(a.ltiles * tile_bytes + fixed);
  if (lds_bytes > 64 * 1024) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds_bytes);
    (void)hipGetLastError();
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kWideThreads), lds_bytes, st, c, kp, a);
  return hipGetLastError();
}

}  // namespace laim
