// Device helpers shared by the kernels of the draft step: number formats, cross-lane moves, sorting
// networks, streaming top-K, the Transition of Eq. 3.  Included inside an unnamed namespace.
#pragma once

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float bf16_to_float(uint16_t h) {
  return __uint_as_float((uint32_t)h << 16);
}
__device__ __forceinline__ uint16_t float_to_bf16(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
// max(a, b) for operands that are never NaN, as the single instruction it is (the generic maximum
// first rewrites both operands into canonical form, two more instructions per call).
__device__ __forceinline__ float max_of_numbers(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// Two running maxima in one register: (a, b) rounded towards zero to half precision, packed, and
// the element-wise maximum of two such pairs.  A maximum kept this way is off by less than one
// half-precision unit in the last place (2^-10 relative; below 2^-14 in magnitude: 2^-24
// absolute); half_floor / half_ceil turn it back into a float32 bound on the true maximum from
// below / above.  Values beyond the half range (|x| > 65504) are clamped by the conversion and
// must be detected by the caller (half_out_of_range).
__device__ __forceinline__ uint32_t pack_halves_rtz(float a, float b) {
  auto p = __builtin_amdgcn_cvt_pkrtz(a, b);
  uint32_t r;
  __builtin_memcpy(&r, &p, 4);
  return r;
}
__device__ __forceinline__ uint32_t max_of_half_pairs(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float half_bits_to_float(uint32_t h) {
  const uint16_t x = (uint16_t)h;
  _Float16 f;
  __builtin_memcpy(&f, &x, 2);
  return (float)f;
}
__device__ __forceinline__ float half_floor(float m) { return m - fabsf(m) * 0.0009765625f - 1e-7f; }
__device__ __forceinline__ float half_ceil(float m) { return m + fabsf(m) * 0.0009765625f + 1e-7f; }
__device__ __forceinline__ bool half_out_of_range(float m) {
  return fabsf(m) >= 60000.f && fabsf(m) < INFINITY;
}
// Order-preserving map float -> uint32 (larger float <=> larger integer) and back.
__device__ __forceinline__ uint32_t ordered_bits(float f) {
  uint32_t u = __float_as_uint(f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float unordered_bits(uint32_t o) {
  uint32_t u = (o & 0x80000000u) ? (o ^ 0x80000000u) : ~o;
  return __uint_as_float(u);
}

// ---- cross-lane helpers (wave64) ---------------------------------------------------------
// Orders this wave's LDS traffic: the hardware runs one wave's LDS instructions in issue
// order, so only the compiler has to be kept from moving accesses across this point.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Value of lane (lane ^ M) for a compile-time M.  Distances 1, 2 and 8 are one DPP move
// (quad permutes, rotation by 8 inside a row of 16 lanes); 4 takes the two rotations by 4 and
// 12; 16 and 32 use the gfx950 row / half-wave swaps.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
  if constexpr (M == 1) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
  } else if constexpr (M == 2) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
  } else if constexpr (M == 4) {
    const uint32_t down = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, true);
    const uint32_t up = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x12C, 0xF, 0xF, true);
    return (lane & 4) ? down : up;   // row_ror:4 reads lane-4, row_ror:12 reads lane+4
  } else if constexpr (M == 8) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);
  } else if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (lane & 16) ? r[0] : r[1];
  } else {
    static_assert(M == 32, "lane distance");
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (lane & 32) ? r[0] : r[1];
  }
}

// One compare-exchange step of the bitonic network across lanes at distance LM, for R
// independent sequences at once (independent work hides the cross-lane latency).
template <int NPL, int R, int LM, typename T>
__device__ __forceinline__ void cross_step(T (&key)[R][NPL], int lane, bool keep_max) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
      T other;
      if constexpr (sizeof(T) == 8) {
        const uint32_t lo = lane_xor<LM>((uint32_t)key[r][j], lane);
        const uint32_t hi = lane_xor<LM>((uint32_t)(key[r][j] >> 32), lane);
        other = ((uint64_t)hi << 32) | lo;
      } else {
        other = lane_xor<LM>(key[r][j], lane);
      }
      const bool gt = key[r][j] > other;
      key[r][j] = (gt == keep_max) ? key[r][j] : other;
    }
}

// Bitonic sort of R sequences of 64*NPL keys (64- or 32-bit unsigned), NPL per lane, descending
// in position p = lane*NPL + j.
template <int NPL, int R, typename T = uint64_t>
__device__ __forceinline__ void sort_desc(T (&key)[R][NPL]) {
  const int lane = threadIdx.x & 63;
  constexpr int N = 64 * NPL;
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int dist = k >> 1; dist >= 1; dist >>= 1) {
      if (dist < NPL) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NPL; ++j) {
            if ((j & dist) == 0) {
              const int j2 = j | dist;
              // block direction: descending where bit k of the position is clear
              const bool desc = (k < NPL) ? ((j & k) == 0)
                                          : (k == N ? true : ((lane & (k / NPL)) == 0));
              const T a = key[r][j], b = key[r][j2];
              const bool a_gt = a > b;
              const bool swap = desc ? !a_gt : a_gt;
              key[r][j] = swap ? b : a;
              key[r][j2] = swap ? a : b;
            }
          }
      } else {
        const int lm = dist / NPL;
        const bool is_lo = (lane & lm) == 0;
        const bool desc = (k == N) ? true : ((lane & (k / NPL)) == 0);
        const bool keep_max = (is_lo == desc);
        if (lm == 1) cross_step<NPL, R, 1, T>(key, lane, keep_max);
        else if (lm == 2) cross_step<NPL, R, 2, T>(key, lane, keep_max);
        else if (lm == 4) cross_step<NPL, R, 4, T>(key, lane, keep_max);
        else if (lm == 8) cross_step<NPL, R, 8, T>(key, lane, keep_max);
        else if (lm == 16) cross_step<NPL, R, 16, T>(key, lane, keep_max);
        else cross_step<NPL, R, 32, T>(key, lane, keep_max);
      }
    }
  }
}

// Cuts R LDS buffers (R rows) back to their K largest keys, sorted descending at buf[0..):
// rows[r] points at CAP keys of which cnt[r] are in use.  On return cnt[r] = min(cnt[r], K)
// and tau[r] is the K-th largest key (0 while fewer than K are held).  Wave uniform.
template <int CAP, int NPL, int R>
__device__ __forceinline__ void compact_rows_n(uint64_t* const (&rows)[R], int (&cnt)[R],
                                               uint64_t (&tau)[R], int K) {
  const int lane = threadIdx.x & 63;
  uint64_t key[R][NPL];
  wave_sync();
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
      const int e = j * 64 + lane;
      key[r][j] = e < cnt[r] ? rows[r][e] : 0ull;
    }
  sort_desc<NPL, R>(key);
  wave_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int keep = cnt[r] < K ? cnt[r] : K;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
      const int p = lane * NPL + j;
      if (p < keep) rows[r][p] = key[r][j];
    }
    cnt[r] = keep;
  }
  wave_sync();
#pragma unroll
  for (int r = 0; r < R; ++r) tau[r] = (cnt[r] == K) ? rows[r][K - 1] : 0ull;
}

// Picks the smallest network that holds every row (all counts are wave uniform).
template <int CAP, int R>
__device__ __forceinline__ void compact_rows(uint64_t* const (&rows)[R], int (&cnt)[R],
                                             uint64_t (&tau)[R], int K) {
  int most = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) most = cnt[r] > most ? cnt[r] : most;
  if (most <= 64) {
    compact_rows_n<CAP, 1, R>(rows, cnt, tau, K);
  } else if (CAP == 128 || most <= 128) {
    compact_rows_n<CAP, 2, R>(rows, cnt, tau, K);
  } else {
    compact_rows_n<CAP, CAP / 64, R>(rows, cnt, tau, K);
  }
}

// A streaming top-K of 64-bit keys for one wave.  The buffer lives in LDS (CAP keys); keys
// that beat the threshold are appended with a ballot prefix; when fewer than 64 free places
// remain the buffer is sorted and cut back to the K largest, which raises the threshold.
template <int CAP>
struct WaveTopK {
  uint64_t* buf;   // LDS, CAP entries, private to the wave
  int cnt;         // wave uniform
  uint64_t tau;    // keys must be > tau to enter; wave uniform
  int K;

  __device__ __forceinline__ void init(uint64_t* b, int k) {
    buf = b;
    cnt = 0;
    tau = 0;
    K = k;
  }
  // Sort, keep the K largest at buf[0..), update tau.
  __device__ __forceinline__ void compact() {
    uint64_t* const rows[1] = {buf};
    int c[1] = {cnt};
    uint64_t t[1] = {0};
    compact_rows<CAP, 1>(rows, c, t, K);
    cnt = c[0];
    tau = t[0];
  }
  // One key per lane (0 = nothing).  All lanes of the wave must call this together.
  __device__ __forceinline__ void push(uint64_t key) {
    const bool pass = key > tau;
    const uint64_t bal = __ballot(pass);
    if (bal) {
      const int pos = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
      if (pass) buf[pos] = key;
      cnt += __popcll(bal);
      if (cnt > CAP - 64) compact();
    }
  }
};

// ---- the Transition of Eq. 3 ------------------------------------------------------------------
// Eq. 3 with the additive Transition for the K survivors of request b: c' = c_parent + E[code]
// (zero for unused slots); 8 (bf16) or 4 (f32) elements per thread and step.
// lds_in / lds_out (bf16 only, may be NULL): the parents' states [K_in, e] and a second copy of
// the new states [K, e] in LDS, for a caller that runs the next level in the same workgroup; ld:
// elements between their rows (0: e).
template <bool BF16>
__device__ __forceinline__ void update_states(const void* state_in, const void* E, void* state_out,
                                              int b, int K, int K_in, int e,
                                              const int32_t* fin_parent, const int32_t* fin_code,
                                              int tid, int nthreads,
                                              const uint16_t* lds_in = nullptr,
                                              uint16_t* lds_out = nullptr, int ld = 0) {
  ld = ld ? ld : e;
  {
    const int per = e / (BF16 ? 8 : 4);
    for (int idx = tid; idx < K * per; idx += nthreads) {
      const int j = idx / per, t = idx - j * per;
      const int par = fin_parent[j], code = fin_code[j];
      if constexpr (BF16) {
        uint16_t* out = static_cast<uint16_t*>(state_out) + ((int64_t)b * K + j) * e + t * 8;
        uint4 r = uint4{0, 0, 0, 0};
        if (par >= 0) {
          const uint4 ev = load_global_u4(static_cast<const uint16_t*>(E) + (int64_t)code * e + t * 8);
          uint4 sv = uint4{0, 0, 0, 0};
          if (lds_in)
            sv = *reinterpret_cast<const uint4*>(lds_in + par * ld + t * 8);
          else if (state_in)
            sv = load_global_u4(static_cast<const uint16_t*>(state_in) +
                                ((int64_t)b * K_in + par) * e + t * 8);
          const uint32_t ew[4] = {ev.x, ev.y, ev.z, ev.w}, sw[4] = {sv.x, sv.y, sv.z, sv.w};
          uint32_t ow[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float lo = bf16_to_float((uint16_t)ew[u]) + bf16_to_float((uint16_t)sw[u]);
            const float hi = bf16_to_float((uint16_t)(ew[u] >> 16)) +
                             bf16_to_float((uint16_t)(sw[u] >> 16));
            ow[u] = (uint32_t)float_to_bf16(lo) | ((uint32_t)float_to_bf16(hi) << 16);
          }
          r = uint4{ow[0], ow[1], ow[2], ow[3]};
        }
        store_global_u4(out, r);
        if (lds_out) *reinterpret_cast<uint4*>(lds_out + j * ld + t * 8) = r;
      } else {
        float* out = static_cast<float*>(state_out) + ((int64_t)b * K + j) * e + t * 4;
        float4 r = float4{0.f, 0.f, 0.f, 0.f};
        if (par >= 0) {
          const float4 ev = *reinterpret_cast<const float4*>(static_cast<const float*>(E) +
                                                             (int64_t)code * e + t * 4);
          float4 sv = float4{0.f, 0.f, 0.f, 0.f};
          if (state_in)
            sv = *reinterpret_cast<const float4*>(static_cast<const float*>(state_in) +
                                                  ((int64_t)b * K_in + par) * e + t * 4);
          r = float4{ev.x + sv.x, ev.y + sv.y, ev.z + sv.z, ev.w + sv.w};
        }
        *reinterpret_cast<float4*>(out) = r;
      }
    }
  }
}

// Eq. 3 with the recurrent Transition for the K survivors of request b:
// c'[j] = tanh(sum_i U[j][i] c_parent[i] + E[code][j]) (zero for unused slots).  bf16: 16x16
// output tiles (16 survivors x 16 state elements) by v_mfma_f32_16x16x32_bf16, spread over the
// workgroup's waves; the accumulator starts at the code embedding; the A operand is the parent
// state row, the B operand B[k][n] = U[n][k] is 16 contiguous bytes of row n of U.
template <bool BF16>
__device__ __forceinline__ void update_states_rnn(const void* state_in, const void* E, const void* U,
                                                  void* state_out, int b, int K, int K_in, int e,
                                                  const int32_t* fin_parent,
                                                  const int32_t* fin_code, int tid, int nthreads,
                                                  const uint16_t* lds_in = nullptr,
                                                  uint16_t* lds_out = nullptr, int ld = 0) {
  ld = ld ? ld : e;
  if constexpr (BF16) {
    const int lane = tid & 63, wave = tid >> 6, n_waves = nthreads >> 6;
    const int g = lane >> 4, c = lane & 15;
    const int RT = (K + 15) / 16, CT = e / 16, KS = e / 32;
    const uint16_t* Eh = static_cast<const uint16_t*>(E);
    const uint16_t* Uh = static_cast<const uint16_t*>(U);
    const uint16_t* Sh = static_cast<const uint16_t*>(state_in);
    uint16_t* Oh = static_cast<uint16_t*>(state_out);
    for (int t = wave; t < RT * CT; t += n_waves) {
      const int rt = t / CT, ct = t - rt * CT;
      floatx4 acc;
      int code[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = rt * 16 + 4 * g + i;
        code[i] = j < K ? fin_code[j] : -1;
        acc[i] = code[i] >= 0 ? bf16_to_float(as_global(Eh)[(int64_t)code[i] * e + ct * 16 + c]) : 0.f;
      }
      const int ja = rt * 16 + c;
      const int pa = ja < K ? fin_parent[ja] : -1;
      if (Sh || lds_in) {
        for (int ks = 0; ks < KS; ++ks) {
          uint4 av = uint4{0, 0, 0, 0};
          if (pa >= 0) {
            if (lds_in)
              av = *reinterpret_cast<const uint4*>(lds_in + pa * ld + ks * 32 + 8 * g);
            else
              av = load_global_u4(Sh + ((int64_t)b * K_in + pa) * e + ks * 32 + 8 * g);
          }
          const uint4 bv = load_global_u4(Uh + (int64_t)(ct * 16 + c) * e + ks * 32 + 8 * g);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(&av),
                                                        *reinterpret_cast<const bf16x8*>(&bv), acc,
                                                        0, 0, 0);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = rt * 16 + 4 * g + i;
        if (j < K) {
          const uint16_t v = code[i] >= 0 ? float_to_bf16(tanhf(acc[i])) : (uint16_t)0;
          as_global(Oh)[((int64_t)b * K + j) * e + ct * 16 + c] = v;
          if (lds_out) lds_out[j * ld + ct * 16 + c] = v;
        }
      }
    }
  } else {
    const float* Ef = static_cast<const float*>(E);
    const float* Uf = static_cast<const float*>(U);
    const float* Sf = static_cast<const float*>(state_in);
    float* Of = static_cast<float*>(state_out);
    for (int idx = tid; idx < K * e; idx += nthreads) {
      const int j = idx / e, col = idx - j * e;
      const int par = fin_parent[j], code = fin_code[j];
      float r = 0.f;
      if (par >= 0) {
        float acc = Ef[(int64_t)code * e + col];
        if (Sf) {
          const float* srow = Sf + ((int64_t)b * K_in + par) * e;
          const float* urow = Uf + (int64_t)col * e;
          for (int i = 0; i < e; ++i) acc = fmaf(urow[i], srow[i], acc);
        }
        r = tanhf(acc);
      }
      Of[((int64_t)b * K + j) * e + col] = r;
    }
  }
}

