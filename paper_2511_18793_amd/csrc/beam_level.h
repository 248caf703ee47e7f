// All levels of a decode (or one level) for beams of up to 128, bf16: one workgroup per request.
// Included inside the library's unnamed namespace, after beam_args.h, device_common.h, beam_common.h.
#pragma once

constexpr int kGapBins = 256;
constexpr int kGmRow = 8 * 16 + 1;         // region x, group maxima: words per beam

// The fixed part of a workgroup's LDS.
struct alignas(16) BeamShared {
  uint64_t key[2][kBeamMax];    // Eq. 4 indices of the entering / leaving beams
  uint64_t best[kBeamMax];      // exhaustive verification: candidates that are settled
  unsigned long long t64;       // list threshold
  float sp[2][kBeamMax];        // the beams' scores (-inf: empty slot)
  alignas(16) float off[kBeamMax];  // score - log-sum-exp of each entering beam
  alignas(16) float lb[kBeamMax];   // exhaustive verification: lower bound of the beam's K-th logit
  alignas(16) float part[kBeamWaves][kBeamMax];
  alignas(16) uint32_t hist[2][kGapBins];
  alignas(16) uint32_t rank[kBeamThreads];
  uint32_t beam_n[kBeamMax];    // listed candidates per beam
  alignas(16) int wave_n[2][kBeamWaves];  // listed and marked candidates of each wave
  int32_t fin_parent[kBeamMax], fin_code[kBeamMax];
  uint32_t sp_max;              // ordered bits of the best entering score, 0: no beam lives
  int n_list, n_valid, flag, n_rows, n_best;
  int sure;                     // gap bins that hold at most K of all candidates
};

// ---- score thresholds from a histogram of gaps ---------------------------------------------------
// gap = (best parent score) - score >= 0; 32 bins per factor of two from 1/8 on, so that the
// resolution follows the spread of the scores whatever their scale.
constexpr uint32_t kGapBase = 0x3E000000u >> 18;            // bits of 1/8
__device__ __forceinline__ int gap_bin(float gap) {
  const uint32_t u = __float_as_uint(fmaxf(gap, 0.125f)) >> 18;
  const int b = (int)(u - kGapBase);
  return b < kGapBins - 1 ? b : kGapBins - 1;
}
// Counts one score (-inf and what lies beyond the last bin: not counted).
__device__ __forceinline__ void gap_count(uint32_t* hist, float best, float score) {
  const int bin = gap_bin(best - score);
  if (bin < kGapBins - 1) atomicAdd(&hist[bin], 1u);
}
// The score threshold that at least `want` of the values counted in hist reach (-inf: fewer were
// counted).  Every wave gets the result.
__device__ __forceinline__ float gap_threshold(const uint32_t* hist, uint32_t want, float best,
                                               int lane) {
  static_assert(kGapBins == 256, "four bins per lane");
  const uint4 h = *reinterpret_cast<const uint4*>(hist + lane * 4);
  const uint32_t c1 = h.x, c2 = c1 + h.y, c3 = c2 + h.z, mine = c3 + h.w;
  const uint32_t incl = wave_prefix(mine);
  const uint64_t reach = __ballot(incl >= want);
  if (reach == 0ull) return -INFINITY;
  const uint32_t above = incl - mine;
  const int bin = lane * 4 + (above + c1 < want) + (above + c2 < want) + (above + c3 < want);
  const int first = __ffsll((unsigned long long)reach) - 1;
  const int at = __builtin_amdgcn_readlane(bin, first);
  const float gap = __uint_as_float((uint32_t)(at + 1 + (int)kGapBase) << 18);
  return best - gap - 1e-5f * (fabsf(best) + gap + 1.f);
}
// How many leading bins together hold at most `most` of the counted values.
__device__ __forceinline__ int gap_bins_within(const uint32_t* hist, uint32_t most, int lane) {
  const uint4 h = *reinterpret_cast<const uint4*>(hist + lane * 4);
  const uint32_t c1 = h.x, c2 = c1 + h.y, c3 = c2 + h.z, mine = c3 + h.w;
  const uint32_t incl = wave_prefix(mine);
  const uint64_t past = __ballot(incl > most);
  if (past == 0ull) return kGapBins - 1;
  const uint32_t above = incl - mine;
  const int bin = lane * 4 + (above + c1 <= most) + (above + c2 <= most) + (above + c3 <= most);
  return __builtin_amdgcn_readlane(bin, __ffsll((unsigned long long)past) - 1);
}
__device__ __forceinline__ float pick4(float a, float b, float c, float d, int k) {
  const float lo = (k & 1) ? b : a, hi = (k & 1) ? d : c;
  return (k & 2) ? hi : lo;
}

// One workgroup of eight waves per request runs all levels; beams, scores and states stay in LDS.
//
// What bounds it: at large shapes (B K T_l logits per level) the matrix and vector instructions of
// the sweeps, which overlap only in part and run at the clock the chip sustains under both; at small
// ones the length of the chain of short steps between barriers (a wave issues one instruction in
// about five cycles, so what counts is how many there are on that chain).
//
// The waves split the codes, not the beams: wave w takes the column tiles w, w + 8, ... of 16 codes for
// all of the request's beams, whose states it holds in registers as MFMA operands.  The packed part
// of W_l then crosses L2 -> CU once per sweep and goes straight into registers (no staging through
// LDS, no barrier inside a sweep), and the row tiles' accumulation chains are independent of each
// other.  A level:
//   sweep 1   z = A_l + c W_l; per lane and beam the sum of exponentials and the largest logit
//   threshold every (lane, beam) maximum is the logit of a candidate of its own, so a score that
//             enough of those maxima reach bounds the request's K-th best from below: two histograms
//             of score gaps (of the lanes' best, then of the maxima at or above the first result)
//   sweep 2   the logits again; what reaches the threshold is listed as sort keys (score, parent,
//             code), about 1.3 K of them
//   places    every listed candidate against every other one, outputs, Transition
// With a set the threshold is set for 2 K candidates and the listed ones are looked up in the table
// (one per thread).  If fewer than K of them are items, all of the beams' K best codes have to be
// considered: sweep 3 lists only what has its bit set in the set's prefilter and can be among its
// beam's K best (see below), a few codes per beam.
// W operands and user part of the column tiles requested ahead
template <int KST, int RT>
struct BeamTiles {
  // matrix tiles in the pipeline ahead of the one in the vector units, and column tiles requested ahead
  static constexpr int kAhead = RT == 1 && KST > 2 ? 1 : 2;
  static constexpr int NB = RT == 1 ? kAhead + 1 : KST > 4 || RT >= 5 || RT == 2 ? 2 : 3;
  uint4 w[NB][KST];
  float a0[NB];
};
// The operands of a level's logits and the loop that forms them; a wave's view.
template <int KST, int RT>
struct BeamSweep {
  static constexpr bool kExact = KST <= 4;                 // e == 32 KST
  static constexpr bool kFaRegs = RT * KST <= (KST > 4 ? 8 : 32);
  static constexpr int NB = BeamTiles<KST, RT>::NB;
  int lane, g, c, wave, n_mine, KS, K_in, e, state_ld;
  const uint16_t* states;                                  // LDS copy of the states, or NULL
  const uint16_t* state_in;                                // the request's states in global memory, or NULL
  const float* Arow;
  const uint16_t* Wl;
  uint4 fa[kFaRegs ? RT : 1][kFaRegs ? KST : 1];           // the beams' states as MFMA operands
  uint4 (&w)[NB][KST];
  float (&a0)[NB];

  // (states: LDS copy of the entering states, or NULL)
  __device__ __forceinline__ BeamSweep(BeamTiles<KST, RT>& t, const BeamLevel& v, const uint16_t* states_,
                                       int ld, int e_, int b) : w(t.w), a0(t.a0) {
    lane = fresh((int)threadIdx.x) & 63;
    wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    g = lane >> 4;
    c = lane & 15;
    e = e_;
    KS = kExact ? KST : e >> 5;
    K_in = v.K_in;
    state_ld = ld;
    states = states_;
    state_in = v.state_in ? static_cast<const uint16_t*>(v.state_in) + (int64_t)b * K_in * e : nullptr;
    Arow = v.A + (int64_t)b * v.V;
    Wl = static_cast<const uint16_t*>(v.Wbeam) + lane * 8;
    const int n_ct = v.V >> 4;
    n_mine = wave < n_ct ? (n_ct - wave + kBeamWaves - 1) / kBeamWaves : 0;
  }
  __device__ __forceinline__ uint4 load_fa(int par, int ks) const {   // 16 bytes of beam par's state
    uint4 x = uint4{0, 0, 0, 0};
    if (par < K_in && (kExact || ks < KS)) {
      if (states)
        x = *reinterpret_cast<const uint4*>(states + par * state_ld + ks * 32 + 8 * g);
      else if (state_in)
        x = load_global_u4(state_in + par * e + ks * 32 + 8 * g);
    }
    return x;
  }
  __device__ __forceinline__ void load_beams() {
    if constexpr (kFaRegs) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) fa[rt][ks] = load_fa(16 * rt + c, ks);
    }
  }
  __device__ __forceinline__ void load_w(int k, int j) {   // the wave's column tile j into buffer k
    const int ct = wave + kBeamWaves * j;
    a0[k] = as_global(Arow)[ct * 16 + c];
    const uint16_t* p = Wl + (int64_t)ct * KS * 512;
#pragma unroll
    for (int ks = 0; ks < KST; ++ks) {
      if (kExact || ks < KS) w[k][ks] = load_global_u4(p + ks * 512);
      else w[k][ks] = uint4{0, 0, 0, 0};
    }
  }
  __device__ __forceinline__ floatx4 link(floatx4 acc, int k, int rt, int ks) const {
    uint4 x;
    if constexpr (kFaRegs) x = fa[rt][ks];
    else x = load_fa(16 * rt + c, ks);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(&x),
                                                   *reinterpret_cast<const bf16x8*>(&w[k][ks]), acc, 0,
                                                   0, 0);
  }
  __device__ __forceinline__ floatx4 start(int k) const { return floatx4{a0[k], a0[k], a0[k], a0[k]}; }
  // The W operands of the wave's first NB column tiles are in w when a sweep starts and again when it
  // ends, so that the next sweep does not begin with a round trip to L2.
  __device__ __forceinline__ int next_tile(int j, int k) const { return j + NB < n_mine ? j + NB : k < n_mine ? k : 0; }
  __device__ __forceinline__ void first_tiles() {
    if (n_mine == 0) {                                     // fewer than eight column tiles: nothing is used
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        a0[k] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) w[k][ks] = uint4{0, 0, 0, 0};
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) load_w(k, k < n_mine ? k : 0);
  }
  // piece(j, ct, rt, i, z) for i = 0..3 of every tile: z, the lane's four logits of row tile rt (beams
  // 16 rt + 4 g + i) and column tile ct (code 16 ct + c); j counts the wave's column tiles.  The
  // matrix instructions of the tile after the next one (or of the next one) are issued between the four pieces of vector
  // work on the current one, so that no vector instruction waits for the end of a chain.
  template <class Piece>
  __device__ __forceinline__ void stream(Piece piece) {
    constexpr int kAhead = BeamTiles<KST, RT>::kAhead;
    floatx4 z0 = start(0), z1 = start(1 / RT);
#pragma unroll
    for (int ks = 0; ks < KST; ++ks) {
      z0 = link(z0, 0, 0, ks);
      if (kAhead > 1) z1 = link(z1, 1 / RT, 1 % RT, ks);
    }
#pragma unroll 1
    for (int j0 = 0; j0 < n_mine; j0 += NB) {
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const int j = j0 + k;
        if (j < n_mine) {
          const int ct = wave + kBeamWaves * j;
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const int kn = (k + (rt + kAhead) / RT) % NB, rn = (rt + kAhead) % RT;
            floatx4 zn = start(kn);
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
              zn = link(zn, kn, rn, ks);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if ((i * KST) / 4 == ks) piece(j, ct, rt, i, z0);
              __builtin_amdgcn_sched_barrier(0);
            }
            if (rt == RT - 1) load_w(k, next_tile(j, k));
            z0 = kAhead > 1 ? z1 : zn;
            z1 = zn;
          }
        }
      }
    }
  }
};

// ---- exhaustive verification: every beam's K best codes ----
// Only codes whose bit is set in the set's prefilter can be items, and only logits at or above a lower
// bound of the beam's K-th largest can be among its K best: sweep 3 lists what meets both (a few per
// beam), the table decides which of them are items, and the items that can still make the request's
// K best are checked for their place inside their beam: sixteen at a time, each as a row of one
// matrix tile, by counting the beam's better codes.  Returns how many candidates are in s.best.
// (A function of its own: its registers and code stay out of the common path.)
extern __shared__ __align__(16) uint8_t beam_lds[];
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uniform(uint64_t x) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32;
}
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
  return reinterpret_cast<T*>(uniform((uint64_t)reinterpret_cast<uintptr_t>(p)));
}
// (arguments arrive in vector registers; all of them are the same for the whole workgroup)
template <int KST, int RT>
__device__ __forceinline__ int beam_exhaustive(
    const void* state_in, const void* Wbeam, const float* A, const uint64_t* slots, uint64_t n_buckets,
    const uint64_t* filter, uint64_t n_blocks, uint64_t mult_last, int K_in_, int V_, int K_, int e_,
    int state_at_, int state_ld_, int b_, int cur_, int x_off, int list_off, int status_off,
    int mask_in_lds) {
  BeamLevel v;
  v.state_in = uniform(state_in);
  v.Wbeam = uniform(Wbeam);
  v.A = uniform(A);
  v.set = SetView{uniform(slots), uniform(n_buckets), uniform(filter), uniform(n_blocks), uniform(mult_last)};
  v.K_in = uniform(K_in_);
  v.V = uniform(V_);
  struct {
    int K, e, x_off, list_off, status_off, mask_in_lds;
  } a = {uniform(K_), uniform(e_), uniform(x_off), uniform(list_off), uniform(status_off),
         uniform(mask_in_lds)};
  const int state_at = uniform(state_at_), state_ld = uniform(state_ld_), b = uniform(b_),
            cur = uniform(cur_);
  BeamShared& s = *reinterpret_cast<BeamShared*>(beam_lds);
  uint64_t* const list = reinterpret_cast<uint64_t*>(beam_lds + a.list_off);
  constexpr int NB = BeamSweep<KST, RT>::NB;
  const int tid = fresh((int)threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int V = v.V, K = a.K, K_in = v.K_in;
  const int n_ct = V >> 4;
  float* const gm_dump = reinterpret_cast<float*>(beam_lds + a.x_off);
  uint16_t* const mask = reinterpret_cast<uint16_t*>(beam_lds + a.x_off);
  uint8_t* const lds = beam_lds;
  const uint64_t* const keys = s.key[cur];
  uint64_t mine[kBeamMaxPer];
  int n;
  BeamTiles<KST, RT> tiles;
  BeamSweep<KST, RT> sw(tiles, v, state_at >= 0 ? reinterpret_cast<const uint16_t*>(beam_lds + state_at) : nullptr,
                        state_ld, a.e, b);
  const int n_mine = sw.n_mine;
  const int sure = s.sure;
  const float best_sp = unordered_bits(s.sp_max);
  constexpr int PER = kBeamMaxPer + 1;                   // a full list and what was settled before
  const bool use_lb = K_in * V > 16384;                  // below that the bits alone are enough
  __syncthreads();
  if (use_lb) {
    // lower bound: a bisection of the 128 group maxima for their K-th largest
#pragma unroll 1
    for (int q = wave * 4; q < 16 * RT; q += 4 * kBeamWaves) {
      float x0[4], x1[4], lo[4], hi[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x0[r] = gm_dump[(q + r) * kGmRow + lane];
        x1[r] = gm_dump[(q + r) * kGmRow + 64 + lane];
        lo[r] = -wave_max_f(-fminf(x0[r], x1[r]), lane);
        hi[r] = wave_max_f(fmaxf(x0[r], x1[r]), lane);
      }
#pragma unroll 1
      for (int step = 0; step < 9; ++step) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float mid = 0.5f * (lo[r] + hi[r]);
          const bool enough = __popcll(__ballot(x0[r] >= mid)) + __popcll(__ballot(x1[r] >= mid)) >= K;
          lo[r] = enough ? mid : lo[r];
          hi[r] = enough ? hi[r] : mid;
        }
      }
      if (lane == 0)
        *reinterpret_cast<float4*>(&s.lb[q]) = float4{lo[0], lo[1], lo[2], lo[3]};
    }
  } else if (tid < 16 * RT) {
    s.lb[tid] = -INFINITY;
  }
  __syncthreads();                                       // (the maxima make room for the bits)
  // prefilter bits: mask[ct * 16 RT + r] = the 16 codes of tile ct of beam r; a lane reads those of its
  // four beams at once
  if (a.mask_in_lds) {
    const int n_w = (V + 63) >> 6;
#pragma unroll 4
    for (int x = tid; x < 16 * RT * n_w; x += kBeamThreads) {
      const int par = x / n_w, wi = x - par * n_w;
      uint64_t bits = 0ull;
      if (par < K_in && keys[par] != kEmpty)
        bits = v.set.filter ? *(global_ptr<const uint64_t>)(v.set.filter +
                                                            filter_word(keys[par], (uint32_t)wi << 6,
                                                                        v.set.n_blocks))
                            : ~0ull;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (4 * wi + q < n_ct) mask[(4 * wi + q) * RT * 16 + par] = (uint16_t)(bits >> (16 * q));
    }
  }
  uint8_t* const status = reinterpret_cast<uint8_t*>(lds + a.status_off);   // 0 open, 1 in, 2 out
  uint16_t* const open_at = reinterpret_cast<uint16_t*>(lds + a.status_off + kBeamStatusBytes / 2);
  uint64_t* const part = list + wave * kPart;
  const int n_units = ((n_ct + kBeamWaves - 1) / kBeamWaves) * RT;
  int u0 = 0, u1 = n_units, nb = 0;
#pragma unroll 1
  while (u0 < n_units) {
    const int tid = fresh((int)threadIdx.x), lane = tid & 63, g = lane >> 4, c = lane & 15;
    int wn;
    __syncthreads();
    sw.first_tiles();
    sw.load_beams();
    {
      float bound[RT][4];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * rt + 4 * g + i;
          bound[rt][i] = s.off[row] == -INFINITY ? INFINITY : s.lb[row];
        }
      wn = 0;
      sw.stream([&](int j, int ct, int rt, int i, const floatx4& z) {
        if (i != 3) return;
        const int unit = j * RT + rt;
        if (unit < u0 || unit >= u1) return;
        uint32_t hit = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) hit |= z[k] >= bound[rt][k] ? 1u << k : 0u;
        if (a.mask_in_lds) {
          const uint2 w = *reinterpret_cast<const uint2*>(mask + ct * RT * 16 + rt * 16 + 4 * g);
          hit &= ((w.x >> c) & 1u) | ((w.x >> (c + 15)) & 2u) | (((w.y >> c) & 1u) << 2) | (((w.y >> (c + 15)) & 2u) << 2);
        }
        if (__ballot(hit != 0u) == 0ull) return;
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
          bool in = (hit >> k) & 1u;
          uint64_t p = __ballot(in);
          if (p == 0ull) continue;
          const int par = 16 * rt + 4 * g + k;
          const uint32_t code = (uint32_t)(ct * 16 + c);
          if (!a.mask_in_lds && v.set.filter) {
            if (in)
              in = (*(global_ptr<const uint64_t>)(v.set.filter +
                                                  filter_word(keys[par], code, v.set.n_blocks)) >>
                    (code & 63)) & 1ull;
            p = __ballot(in);
          }
          const float score = s.off[par] + pick4(z[0], z[1], z[2], z[3], k);
          part_push(part, wn, p, in, beam_entry(score, par, code));
        }
      });
    }
    if (lane == 0) s.wave_n[0][wave] = wn;
    const int held = wn < kPart ? wn : kPart;
    part_mine(part, held, lane, mine);
    const uint32_t ok = probe_mine(v.set, keys, held, lane, mine);
    const int marked = count_marked(ok);
    if (lane == 0) s.wave_n[1][wave] = marked;
    __syncthreads();
    if (wave_counts(s.wave_n[0], wave).most > kPart) {   // the codes in two halves, then
      u1 = u0 + (u1 - u0 > 1 ? (u1 - u0) / 2 : 1);       // (one unit: 256 candidates per wave, which fit)
      continue;
    }
    const WaveCounts found = wave_counts(s.wave_n[1], wave);
    pack_marked(list, found.before, ok, mine);
    const int n_new = found.total;
    n = n_new + nb;
    if (tid < nb) list[n_new + tid] = s.best[tid];       // what earlier rounds settled
    __syncthreads();
    // Which of them are among their beam's K best: decided for those above a floor, which about K + 32
    // of them reach at first and twice as many whenever fewer than K of those are in.
    for (int i = tid; i < n; i += kBeamThreads) status[i] = i >= n_new || gap_bin(best_sp - entry_score(list[i])) < sure ? 1 : 0;
    int want = K + 32;
    float floor = INFINITY;
#pragma unroll 1
    for (;;) {
      const int tid = fresh((int)threadIdx.x), lane = tid & 63, g = lane >> 4, c = lane & 15;
      if (floor == INFINITY) {                             // a new floor
        if (tid < kGapBins) s.hist[0][tid] = 0u;
        lds_barrier();
        for (int i = tid; i < n; i += kBeamThreads) gap_count(s.hist[0], best_sp, entry_score(list[i]));
        lds_barrier();
        floor = gap_threshold(s.hist[0], (uint32_t)want, best_sp, lane);
      }
      if (tid == 0) s.n_rows = s.n_best = 0;
      s.rank[tid] = 0u;
      lds_barrier();
      int in = 0;
#pragma unroll 1
      for (int i0 = 0; i0 < n; i0 += kBeamThreads) {
        const int i = i0 + tid;
        const int st = i < n && entry_score(list[i]) >= floor ? (int)status[i] : 2;
        in += __popcll(__ballot(st == 1));
        if (st == 0) {
          const int at = atomicAdd(&s.n_rows, 1);
          if (at < kBeamThreads) open_at[at] = (uint16_t)i;
        }
      }
      if (lane == 0 && in) atomicAdd(&s.n_best, in);
      lds_barrier();
      const int n_open = s.n_rows < kBeamThreads ? s.n_rows : kBeamThreads, n_in = s.n_best;
      lds_barrier();
      if (n_open == 0) {
        if (n_in >= K || floor == -INFINITY) break;
        want = 2 * want;
        floor = INFINITY;
        continue;
      }
      // sixteen (or 32) at a time: the rows of matrix tiles against all codes, the waves' counts added up
      constexpr int NR = KST <= 4 && RT > 2 ? 2 : 1;
#pragma unroll 1
      for (int q = 0; q < n_open; q += 16 * NR) {
        uint4 fb[NR][KST];
        float off[NR][4], thr[NR][4];
        int code[NR][4];
        uint32_t cnt[NR][4];
#pragma unroll
        for (int t = 0; t < NR; ++t) {
          const int at_c = q + 16 * t + c;
          const int par_c = at_c < n_open ? entry_parent(list[open_at[at_c]]) : K_in;
#pragma unroll
          for (int ks = 0; ks < KST; ++ks) fb[t][ks] = sw.load_fa(par_c, ks);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = q + 16 * t + 4 * g + i;
            const uint64_t er = list[open_at[r < n_open ? r : q]];
            off[t][i] = s.off[entry_parent(er)];
            thr[t][i] = entry_score(er);
            code[t][i] = (int)entry_code(er);
            cnt[t][i] = 0u;
          }
        }
        // (the wave's first NB tiles are in w when this starts and again when it ends; no branch may
        // come between a matrix instruction and the first use of what it gives: the compiler then
        // leaves out the wait on one of the two ways)
#pragma unroll 1
        for (int j0 = 0; j0 < n_mine; j0 += NB) {
#pragma unroll
          for (int k = 0; k < NB; ++k) {
            const int j = j0 + k;
            if (j < n_mine) {
              const int ct = wave + kBeamWaves * j;
              floatx4 z[NR];
#pragma unroll
              for (int t = 0; t < NR; ++t) z[t] = sw.start(k);
#pragma unroll
              for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                for (int t = 0; t < NR; ++t)
                  z[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                      *reinterpret_cast<const bf16x8*>(&fb[t][ks]),
                      *reinterpret_cast<const bf16x8*>(&sw.w[k][ks]), z[t], 0, 0, 0);
              sw.load_w(k, sw.next_tile(j, k));
#pragma unroll
              for (int t = 0; t < NR; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const float sc = off[t][i] + z[t][i];
                  cnt[t][i] += (uint32_t)(sc > thr[t][i]) |
                               ((uint32_t)(sc == thr[t][i]) & (uint32_t)(ct * 16 + c < code[t][i]));
                }
            }
          }
        }
#pragma unroll
        for (int t = 0; t < NR; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t sum = row_sum_u(cnt[t][i]);
            const int r = q + 16 * t + 4 * g + i;
            if (c == 0 && r < n_open) atomicAdd(&s.rank[r], sum);
          }
      }
      lds_barrier();
      if (tid < n_open) status[open_at[tid]] = s.rank[tid] < (uint32_t)K ? 1 : 2;
      lds_barrier();
    }
    // the best K of those that are in are the best so far
    if (tid == 0) s.n_valid = 0;
    uint32_t keep = 0u;
    uint64_t en[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = tid + u * kBeamThreads;
      en[u] = i < n ? list[i] : 0ull;
      if (i < n && entry_score(en[u]) >= floor && status[i] == 1) keep |= 1u << u;
    }
    lds_barrier();
    pack_list(s, list, keep, en, lane);
    lds_barrier();
    n = s.n_valid;
    rank_list(list, n, K, s.rank, wave, lane, [&](uint64_t e, int r) { s.best[r] = e; });
    if (tid == 0) s.n_best = n < K ? n : K;
    __syncthreads();
    nb = s.n_best;
    u0 = u1;
    u1 = n_units;
  }
  return nb;
}

template <int KST, int RT>
__device__ __forceinline__ void beam_level(BeamShared& s, const BeamArgs& a, const BeamLevel& v,
                                           uint8_t* lds, uint64_t* list, int state_at,
                                           int state_ld, int b, int cur) {
  // (state_at: where in LDS the entering states are, -1: in global memory or none)
  const uint16_t* const states = state_at >= 0 ? reinterpret_cast<const uint16_t*>(lds + state_at) : nullptr;
  const int tid0 = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
#define FRESH_LANE const int tid = fresh(tid0), lane = tid & 63, g = lane >> 4, c = lane & 15; (void)g; (void)c
  const int V = v.V, K = a.K, K_in = v.K_in, e = a.e;
  const bool has_state = states != nullptr || v.state_in != nullptr;
  const bool first_level = K_in == 1 && !has_state;        // the logits are the user part
  const bool verify = v.set.slots != nullptr;
  const float* Arow = v.A + (int64_t)b * V;
  float* const gm_dump = reinterpret_cast<float*>(lds + a.x_off);
  const uint64_t* const keys = s.key[cur];

  BeamTiles<KST, RT> tiles;
  BeamSweep<KST, RT> sw(tiles, v, states, state_ld, e, b);
  const int n_mine = sw.n_mine;

  // ---- sweep 1 ----
  // Exponentials about one reference for the whole level, the first code's user part + 20: sums of the
  // waves then simply add up.  A logit more than 60 above it, or a beam whose sum is lost below it,
  // sends the level through the careful pass.
  const float ref = as_global(Arow)[0] + 20.f;
  const float best_sp = unordered_bits(s.sp_max);          // (0: no beam lives)
  const bool dead = s.sp_max == 0u;
  int want = verify && !first_level ? 2 * K + 8 : K;
  constexpr int NV = 8;
  float zf[NV];                                            // first level: eight codes per thread
  float gm[RT][4];
  {
  FRESH_LANE;
  for (int i = tid; i < 2 * kGapBins; i += kBeamThreads) (&s.hist[0][0])[i] = 0u;
  if (tid < kBeamMax) s.beam_n[tid] = 0u;
  if (tid == 0) {
    s.n_list = 0;
    s.n_valid = 0;
    s.flag = 0;
  }
  }
  if (first_level) {
    FRESH_LANE;
    const float nml = -ref * kLog2e;
    float sum = 0.f, top = -INFINITY;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int code = tid + j * kBeamThreads;
      zf[j] = code < V ? as_global(Arow)[code] : -INFINITY;
      top = fmaxf(top, zf[j]);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) sum += __builtin_amdgcn_exp2f(fmaf(zf[j], kLog2e, nml));
    for (int code = tid + NV * kBeamThreads; code < V; code += kBeamThreads) {
      const float z = as_global(Arow)[code];
      top = fmaxf(top, z);
      sum += __builtin_amdgcn_exp2f(fmaf(z, kLog2e, nml));
    }
    sum = wave_sum_f(sum, lane);
    if (lane == 0) s.part[wave][0] = sum;
    gm[0][0] = top;
    __syncthreads();
    if (top > ref + 60.f) s.flag = 1;
  } else {
    FRESH_LANE;
    sw.first_tiles();
    sw.load_beams();
    float ss[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        gm[rt][i] = -INFINITY;
        ss[rt][i] = 0.f;
      }
    float nml = -ref * kLog2e;
    asm volatile("" : "+v"(nml));                          // (in a vector register, as the fma wants it)
    sw.stream([&](int, int, int rt, int i, const floatx4& z) {
      gm[rt][i] = max_of_numbers(gm[rt][i], z[i]);
      ss[rt][i] += __builtin_amdgcn_exp2f(fmaf(z[i], kLog2e, nml));
    });
    float most = -INFINITY;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        t[i] = row_sum(ss[rt][i]);
        most = fmaxf(most, gm[rt][i]);
      }
      if (c == 0)
        *reinterpret_cast<float4*>(&s.part[wave][16 * rt + 4 * g]) = float4{t[0], t[1], t[2], t[3]};
    }
    if (verify) {
      // the lanes' maxima are wanted again if the verification has to be exhaustive
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          gm_dump[(16 * rt + 4 * g + i) * kGmRow + wave * 16 + c] = gm[rt][i];
    }
    lds_barrier();
    if (most > ref + 60.f) s.flag = 1;
  }
  {
  FRESH_LANE;
  if (tid < kBeamMax) {
    float total = 0.f;
#pragma unroll
    for (int q = 0; q < kBeamWaves; ++q) total += s.part[q][tid];
    const bool live = tid < K_in && keys[tid] != kEmpty;
    if (live && !(total > 1e-25f && total < 1e30f)) s.flag = 1;
    const float lse = ref + __builtin_amdgcn_logf(total) * kLn2;
    s.off[tid] = live ? s.sp[cur][tid] - lse : -INFINITY;
  }
  }
  lds_barrier();
  if (s.flag != 0) {
    FRESH_LANE;
    // careful pass: every beam about its own largest logit, one row tile at a time
    __syncthreads();
    if (first_level) {
      float m = gm[0][0];
      m = wave_max_f(m, lane);
      float sum = 0.f;
      for (int code = tid; code < V; code += kBeamThreads)
        sum += __builtin_amdgcn_exp2f((as_global(Arow)[code] - m) * kLog2e);
      sum = wave_sum_f(sum, lane);
      if (lane == 0) s.part[wave][0] = m > -INFINITY ? m + __builtin_amdgcn_logf(sum) * kLn2 : -INFINITY;
    } else {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        float mref[4], sum[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          mref[i] = row_max(gm[rt][i]);                     // over this wave's codes
          sum[i] = 0.f;
        }
#pragma unroll 1
        for (int j = 0; j < n_mine; ++j) {
          sw.load_w(0, j);
          floatx4 z = sw.start(0);
#pragma unroll
          for (int ks = 0; ks < KST; ++ks) z = sw.link(z, 0, rt, ks);
#pragma unroll
          for (int i = 0; i < 4; ++i) sum[i] += __builtin_amdgcn_exp2f((z[i] - mref[i]) * kLog2e);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          sum[i] = row_sum(sum[i]);
          // as one number, its logarithm: the waves' references differ
          const float l = n_mine ? mref[i] + __builtin_amdgcn_logf(sum[i]) * kLn2 : -INFINITY;
          if (c == 0) s.part[wave][16 * rt + 4 * g + i] = l;
        }
      }
      sw.first_tiles();
    }
    __syncthreads();
    if (tid < (first_level ? 1 : 16 * RT)) {
      float mm = s.part[0][tid], total = 0.f;
#pragma unroll
      for (int q = 1; q < kBeamWaves; ++q) mm = fmaxf(mm, s.part[q][tid]);
#pragma unroll
      for (int q = 0; q < kBeamWaves; ++q)
        total += __builtin_amdgcn_exp2f((s.part[q][tid] - mm) * kLog2e);
      const bool live = tid < K_in && keys[tid] != kEmpty;
      const float lse = mm + __builtin_amdgcn_logf(total) * kLn2;
        s.off[tid] = live ? s.sp[cur][tid] - lse : -INFINITY;
    }
    __syncthreads();
  }

  // ---- score threshold ----
  float tau;
  {
    FRESH_LANE;
    float top = -INFINITY;
    if (first_level) {
      top = gm[0][0] + s.off[0];
    } else {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float4 o = *reinterpret_cast<const float4*>(&s.off[16 * rt + 4 * g]);
        gm[rt][0] += o.x;                                   // from here on: scores
        gm[rt][1] += o.y;
        gm[rt][2] += o.z;
        gm[rt][3] += o.w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (RT > 2) top = max_of_numbers(top, gm[rt][i]);
          else gap_count(s.hist[0], best_sp, gm[rt][i]);
        }
      }
    }
    if (RT > 2 || first_level) gap_count(s.hist[0], best_sp, top);
    lds_barrier();
    tau = gap_threshold(s.hist[0], (uint32_t)want, best_sp, lane);
    if (RT > 2 && !first_level) {                          // (up to two row tiles: all were counted at once)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (gm[rt][i] >= tau) gap_count(s.hist[1], best_sp, gm[rt][i]);
      lds_barrier();
      tau = gap_threshold(s.hist[1], (uint32_t)want, best_sp, lane);
    }
  }
  unsigned long long t64 = tau > -INFINITY ? (unsigned long long)ordered_bits(tau) << 32 : 0ull;

  // ---- sweep 2: list the candidates at or above the threshold, keep what the set holds ----
  uint64_t mine[kBeamMaxPer];
  int n = 0;
  uint64_t* const part = list + wave * kPart;
  bool retried = false;
#pragma unroll 1
  while (!dead) {
    FRESH_LANE;
    const float floor = fmaxf(tau, -3.4e38f);              // (an empty slot's -inf never reaches it)
    const bool by_key = (t64 & 0xFFFFFFFFull) != 0ull;     // the threshold is a candidate, not a score
    int wn = 0;
    // score[k]: candidates (par + k, code)
    auto push = [&](float s0, float s1, float s2, float s3, int par, uint32_t code) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float score = k == 0 ? s0 : k == 1 ? s1 : k == 2 ? s2 : s3;
        uint64_t p = __ballot(score >= floor);
        if (p == 0ull) continue;
        const uint64_t entry = beam_entry(score, par + k, code);
        const bool in = score >= floor && (!by_key || entry >= t64);
        if (by_key) p = __ballot(in);
        part_push(part, wn, p, in, entry);
      }
    };
    if (first_level) {
      const float off = s.off[0];
#pragma unroll 1
      for (int j = 0; wave * 64 + j * kBeamThreads < V; ++j) {
        const int code = tid + j * kBeamThreads;
        const float lo = pick4(zf[0], zf[1], zf[2], zf[3], j), hi = pick4(zf[4], zf[5], zf[6], zf[7], j);
        const float z = code >= V ? -INFINITY : j < NV ? (j < 4 ? lo : hi) : as_global(Arow)[code];
        const float score = off + z;
        push(score, -INFINITY, -INFINITY, -INFINITY, 0, (uint32_t)code);
      }
    } else {
      // (scores are formed here exactly as above, where the threshold comes from: off + logit)
      constexpr bool kOffRegs = RT <= 4;                   // otherwise read from LDS for every tile
      floatx4 off[kOffRegs ? RT : 1];
      if constexpr (kOffRegs) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) off[rt] = *reinterpret_cast<const floatx4*>(&s.off[16 * rt + 4 * g]);
      }
      sw.stream([&](int, int ct, int rt, int i, const floatx4& z) {
        floatx4& o = off[kOffRegs ? rt : 0];
        if (!kOffRegs && i == 0) o = *reinterpret_cast<const floatx4*>(&s.off[16 * rt + 4 * g]);
        if (i != 3) return;
        const float s0 = z[0] + o[0], s1 = z[1] + o[1], s2 = z[2] + o[2], s3 = z[3] + o[3];
        if (__ballot(fmaxf(fmaxf(s0, s1), fmaxf(s2, s3)) >= floor) != 0ull)
          push(s0, s1, s2, s3, 16 * rt + 4 * g, (uint32_t)(ct * 16 + c));
      });
    }
    if (lane == 0) s.wave_n[0][wave] = wn;
    const int held = wn < kPart ? wn : kPart;
    part_mine(part, held, lane, mine);
    uint32_t all = 0u;
#pragma unroll
    for (int u = 0; u < kBeamMaxPer; ++u) all |= lane + 64 * u < held ? 1u << u : 0u;
    lds_barrier();
    const WaveCounts listed = wave_counts(s.wave_n[0], wave);
    n = listed.total;
    if (listed.most > kPart || (n < K && t64 != 0ull && (!verify || first_level))) {
      // Too many: the threshold becomes the r-th best of the first 512 listed ones, r / 512 of which
      // is about the share that is wanted.  K of them reach it, and a quarter of them no longer does,
      // so that this ends.  Too few (rounding at the edge of a bin): no threshold.
      __syncthreads();
      if (listed.most > kPart) {
        if (tid == 0) s.n_list = 0;
        __syncthreads();
        int at = 0;
        if (lane == 0) at = atomicAdd(&s.n_list, held);
        pack_marked(list, __builtin_amdgcn_readfirstlane(at), all, mine);
        __syncthreads();
        const int m = s.n_list < kBeamThreads ? s.n_list : kBeamThreads;   // (more than kPart >= 2 K)
        const int share = (int)((int64_t)m * want / n);
        const int r_th = share > 3 * m / 4 ? 3 * m / 4 : share < K ? K : share;
        const uint64_t me = tid < m ? list[tid] : 0ull;
        int above = 0;
#pragma unroll 4
        for (int j = 0; j + 2 <= m; j += 2) {
          const ulonglong2 o = *reinterpret_cast<const ulonglong2*>(list + j);
          above += (o.x > me) + (o.y > me);
        }
        if ((m & 1) && list[m - 1] > me) ++above;
        if (tid < m && above == r_th - 1) s.t64 = me;
      } else if (tid == 0) {
        s.t64 = 0ull;
      }
      __syncthreads();
      t64 = s.t64;
      tau = t64 ? unordered_bits((uint32_t)(t64 >> 32)) : -INFINITY;
      continue;
    }
    if (!verify) {
      pack_marked(list, listed.before, all, mine);
      lds_barrier();
      break;
    }
#pragma unroll
    for (int u = 0; u < kBeamMaxPer; ++u)
      if ((all >> u) & 1u) atomicAdd(&s.beam_n[entry_parent(mine[u])], 1u);
    uint32_t ok = probe_mine(v.set, keys, held, lane, mine);
    lds_barrier();
    // A beam may only bring its own K best codes.  All candidates at or above the threshold are
    // listed, so the place of one inside its beam is known from the list: looked up (a wave per
    // item) for the items of beams with more than K listed candidates.
    if (__ballot(s.beam_n[lane] > (uint32_t)K || s.beam_n[lane + 64] > (uint32_t)K) != 0ull) {
      uint16_t* const check = reinterpret_cast<uint16_t*>(lds + a.status_off);
      pack_marked(list, listed.before, all, mine);         // entry lane + 64 u: place before + lane + 64 u
      s.rank[tid] = 0u;                                    // bits: items that are not their beam's K best
      if (tid == 0) s.n_list = 0;
      lds_barrier();
#pragma unroll
      for (int u = 0; u < kBeamMaxPer; ++u)
        if (((ok >> u) & 1u) && s.beam_n[entry_parent(mine[u])] > (uint32_t)K)
          check[atomicAdd(&s.n_list, 1)] = (uint16_t)(listed.before + lane + 64 * u);
      lds_barrier();
      const int n_check = s.n_list;
#pragma unroll 1
      for (int q = wave; q < n_check; q += kBeamWaves) {
        const int i = __builtin_amdgcn_readfirstlane((int)check[q]);
        const uint64_t en = list[i];
        const int par = entry_parent(en);
        int better = 0;
#pragma unroll 2
        for (int j = lane; j < n; j += 64) {
          const uint64_t o = list[j];
          better += (int)(o > en) & (int)(entry_parent(o) == par);
        }
        better = (int)__builtin_amdgcn_readlane((int)wave_prefix((uint32_t)better), 63);
        if (lane == 0 && better >= K) atomicOr(&s.rank[i >> 5], 1u << (i & 31));
      }
      lds_barrier();
#pragma unroll
      for (int u = 0; u < kBeamMaxPer; ++u) {
        const int i = listed.before + lane + 64 * u;
        if ((ok >> u) & 1u)
          if ((s.rank[i >> 5] >> (i & 31)) & 1u) ok &= ~(1u << u);
      }
    }
    const int marked = count_marked(ok);
    if (lane == 0) s.wave_n[1][wave] = marked;
    lds_barrier();
    const WaveCounts found = wave_counts(s.wave_n[1], wave);
    const int m = found.total;
    if (m >= K || t64 == 0ull || first_level) {            // enough, or everything was listed
      pack_marked(list, found.before, ok, mine);
      lds_barrier();
      n = m;
      break;
    }
    // Too few.  The bins of gaps that hold at most K of all candidates (these are surely among their
    // beam's K best), and how many of those after them are in the set.
    if (tid < kGapBins) s.hist[0][tid] = s.hist[1][tid] = 0u;
    lds_barrier();
#pragma unroll
    for (int u = 0; u < kBeamMaxPer; ++u)
      if ((all >> u) & 1u) gap_count(s.hist[0], best_sp, entry_score(mine[u]));
    lds_barrier();
    const int sure = n > K ? gap_bins_within(s.hist[0], (uint32_t)K, lane) : 0;
    uint32_t low = 0u;
#pragma unroll
    for (int u = 0; u < kBeamMaxPer; ++u)
      low |= ((ok >> u) & 1u) && gap_bin(best_sp - entry_score(mine[u])) >= sure ? 1u << u : 0u;
    const int low_n = count_marked(low);
    if (lane == 0) s.wave_n[1][wave] = low_n;
    if (tid == 0) s.sure = sure;
    lds_barrier();
    const int m_low = wave_counts(s.wave_n[1], wave).total;
    if (tid < kBeamMax) s.beam_n[tid] = 0u;
    // where they are not rare a longer list will do
    const int more = m_low > 0 && n > K ? n + (int)((int64_t)(K - m) * (n - K) / m_low) * 3 / 2 + 64
                                        : kBeamList;
    if (retried || more > kBeamList / 2) {
      n = -1;
      break;
    }
    retried = true;
    want = more;
#pragma unroll 1
    for (int q = 0; q < 4 * RT; ++q) {
      const int row = 4 * (4 * (q >> 2) + g) + (q & 3);
      gap_count(s.hist[1], best_sp, gm_dump[row * kGmRow + wave * 16 + c] + s.off[row]);
    }
    lds_barrier();
    tau = gap_threshold(s.hist[1], (uint32_t)want, best_sp, lane);
    t64 = tau > -INFINITY ? (unsigned long long)ordered_bits(tau) << 32 : 0ull;
  }

  if (n < 0) {
    n = beam_exhaustive<KST, RT>(v.state_in, v.Wbeam, v.A, v.set.slots, v.set.n_buckets, v.set.filter,
                                 v.set.n_blocks, v.set.mult_last, K_in, V, K, e, state_at, state_ld, b,
                                 cur, (int)a.x_off, (int)a.list_off, (int)a.status_off, a.mask_in_lds);
    list = s.best;
  }

  // ---- places, outputs ----
  FRESH_LANE;
  const int nxt = cur ^ 1;
  const int cnt = n < K ? n : K;
  lds_barrier();                                           // (everybody has read sp_max by now)
  if (tid == 0) s.sp_max = 0u;
  if (n > kBeamThreads) lds_barrier();                     // (otherwise rank_list begins with one)
  rank_list(list, n, K, s.rank, wave, lane, [&](uint64_t en, int r) {
    const int par = entry_parent(en);
    const uint32_t code = entry_code(en);
    const float score = entry_score(en);
    const uint64_t key = keys[par] + (uint64_t)code * v.mult;
    const int64_t o = (int64_t)b * K + r;
    as_global(v.key_out)[o] = key;
    as_global(v.score_out)[o] = score;
    as_global(v.parent_out)[o] = par;
    as_global(v.code_out)[o] = (int32_t)code;
    s.key[nxt][r] = key;
    s.sp[nxt][r] = score;
    s.fin_parent[r] = par;
    s.fin_code[r] = (int32_t)code;
    if (r == 0) s.sp_max = ordered_bits(score);
  });
  for (int r = cnt + tid; r < K; r += kBeamThreads) {
    const int64_t o = (int64_t)b * K + r;
    as_global(v.key_out)[o] = kEmpty;
    as_global(v.score_out)[o] = -INFINITY;
    as_global(v.parent_out)[o] = -1;
    as_global(v.code_out)[o] = -1;
    s.key[nxt][r] = kEmpty;
    s.sp[nxt][r] = -INFINITY;
    s.fin_parent[r] = -1;
    s.fin_code[r] = -1;
  }
  if (tid == 0 && v.count_out) as_global(v.count_out)[b] = cnt;
}

#undef FRESH_LANE

template <int KST, int RT>
__global__ __launch_bounds__(kBeamThreads, RT <= 2 && KST <= 4 ? 4 : 2) void beam_kernel(BeamArgs a) {
  BeamShared& s = *reinterpret_cast<BeamShared*>(beam_lds);
  uint64_t* const list = reinterpret_cast<uint64_t*>(beam_lds + a.list_off);
  const int tid = threadIdx.x;
  const int b = blockIdx.x, K = a.K, e = a.e;
  const int ld = e + 8;                                    // padded rows: operand reads without conflicts
  // the entering beams of the first level
  {
    const BeamLevel& v = a.lv[0];
    if (tid == 0) s.sp_max = 0u;
    __syncthreads();
    if (tid < kBeamMax) {
      uint64_t key = kEmpty;
      float sp = -INFINITY;
      if (tid < v.K_in) {
        key = v.key_in ? as_global(v.key_in)[(int64_t)b * v.K_in + tid] : 0ull;
        if (key != kEmpty) sp = v.score_in ? as_global(v.score_in)[(int64_t)b * v.K_in + tid] : 0.f;
      }
      s.key[0][tid] = key;
      s.sp[0][tid] = sp;
      if (key != kEmpty) atomicMax(&s.sp_max, ordered_bits(sp));
    }
    __syncthreads();
  }
  int cur = 0;
  int state_at = -1;                                       // the entering states' place in LDS
#pragma unroll 1
  for (int l = 0; l < a.L; ++l) {
    const BeamLevel& v = a.lv[l];
    beam_level<KST, RT>(s, a, v, beam_lds, list, state_at, ld, b, cur);
    cur ^= 1;
    const int tid = fresh((int)threadIdx.x);
    if (v.state_out) {
      lds_barrier();
      const bool carry = a.state_bufs > 0 && l + 1 < a.L;
      const uint16_t* in = a.state_bufs > 1 && state_at >= 0
                               ? reinterpret_cast<const uint16_t*>(beam_lds + state_at) : nullptr;
      const int second = a.state_off + K * ld * 2;
      const int out_at = a.state_bufs > 1 && state_at == (int)a.state_off ? second : (int)a.state_off;
      uint16_t* out = carry ? reinterpret_cast<uint16_t*>(beam_lds + out_at) : nullptr;
      if (v.transition == NEZHA_TRANSITION_RNN)
        update_states_rnn<true>(v.state_in, v.E, v.U, v.state_out, b, K, v.K_in, e, s.fin_parent,
                                s.fin_code, tid, kBeamThreads, in, out, ld);
      else
        update_states<true>(v.state_in, v.E, v.state_out, b, K, v.K_in, e, s.fin_parent, s.fin_code,
                            tid, kBeamThreads, in, out, ld);
      state_at = carry ? out_at : -1;
      if (a.state_bufs < 2) __threadfence_block();         // the global copy is read back
    } else {
      state_at = -1;
    }
    if (a.state_bufs < 2) __syncthreads();
    else lds_barrier();
  }
}
