// float32: all levels of a decode (or one level) for requests whose logits fit in LDS: one workgroup per
// request.  Included inside the library's unnamed namespace, after beam_args.h, device_common.h and
// beam_common.h.
#pragma once

// One workgroup of eight waves per request.  A level is a chain of short steps, each of them a few
// hundred cycles between two barriers; what the kernel costs is the number of those steps, the
// instructions in them and their latency, not memory (a request's part of W_l comes from L2) and
// not arithmetic.  So the logits are formed once, into LDS, and everything after works on rows:
//   1. logits: wave w forms the column tiles w, w + 8, ... of all the request's beams by MFMA (the
//      user part is the accumulators' start value) and puts them into the LDS tile [K_in][T_l];
//      with one entering beam and no state (level 1) the user part is copied.
//   2. rows: a wave takes whole beams (w, w + 8, ...): log-sum-exp by reductions over its lanes, and
//      each lane's best score over its beams.
//   3. threshold: at least K candidates reach the K-th largest lane best of any one wave, and also
//      the smallest of the waves' q-th largest, q = ceil(K / waves with beams); the larger of the
//      two is taken (a bisection of ordered bits by ballots: a few scalar instructions a step).
//   4. list: candidates at or above it, as sort keys (score, parent, code), about 2 to 5 K of them.
//   5. where a set is consulted, instead of 3 and 4: each beam is cut to its K best codes (the K-th
//      largest logit by a bisection of its bits, counting by ballots), those of them whose bit is set
//      in the set's prefilter (a few per beam) are listed and looked up in the table, one per thread.
//   6. places by counting (every candidate against every other), outputs, Transition.
struct alignas(16) DecodeShared {
  uint64_t key[2][kBeamMax];
  unsigned long long t64;
  float sp[2][kBeamMax];
  float lse[kBeamMax];
  uint32_t rank[kBeamThreads];
  int32_t fin_parent[kBeamMax], fin_code[kBeamMax];
  uint32_t bound_k[kBeamWaves], bound_q[kBeamWaves];
  int n_list, n_valid;
};

// The want-th largest (1 <= want <= 64) of the wave's 64 values, rounded down to its upper `bits`
// bits; 0 if fewer than want values are nonzero.
__device__ __forceinline__ uint32_t wave_kth(uint32_t x, int want, int bits) {
  uint32_t t = 0;
#pragma unroll 1
  for (int bit = 31; bit > 31 - bits; --bit) {
    const uint32_t cand = t | (1u << bit);
    if (__popcll(__ballot(x >= cand)) >= want) t = cand;
  }
  return t;
}

// The word of the set's prefilter that holds the bit (code & 63) of prefix's code (all ones: no filter).
__device__ __forceinline__ uint64_t filter_bits(const SetView& set, uint64_t prefix, int code) {
  if (!set.filter) return ~0ull;
  return *(global_ptr<const uint64_t>)(set.filter + filter_word(prefix, (uint32_t)code, set.n_blocks));
}

template <int KST, int RT>
__global__ __launch_bounds__(kBeamThreads, RT * KST <= 16 ? 4 : 2) void decode_lds_kernel(BeamArgs a) {
  extern __shared__ __align__(16) uint8_t decode_lds[];
  DecodeShared& s = *reinterpret_cast<DecodeShared*>(decode_lds);
  uint64_t* const list = reinterpret_cast<uint64_t*>(decode_lds + a.list_off);
  float* const zt = reinterpret_cast<float*>(decode_lds + a.x_off);      // [K_in][V + 4]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int b = blockIdx.x, K = a.K, e = a.e;
  const int KS = e >> 2;
  {
    const BeamLevel& v = a.lv[0];
    if (tid < kBeamMax) {
      uint64_t key = kEmpty;
      float sp = -INFINITY;
      if (tid < v.K_in) {
        key = v.key_in ? as_global(v.key_in)[(int64_t)b * v.K_in + tid] : 0ull;
        if (key != kEmpty) sp = v.score_in ? as_global(v.score_in)[(int64_t)b * v.K_in + tid] : 0.f;
      }
      s.key[0][tid] = key;
      s.sp[0][tid] = sp;
    }
  }
  int cur = 0;
#pragma unroll 1
  for (int l = 0; l < a.L; ++l) {
    const BeamLevel& v = a.lv[l];
    const int V = v.V, K_in = v.K_in, Vp = V + 4;
    const float* Arow = v.A + (int64_t)b * V;
    const bool verify = v.set.slots != nullptr;
    // ---- 1. logits ----
    if (v.state_in) {
      const int n_ct = V >> 4;
      float fa[RT][KST];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int r = 16 * rt + c;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {
          fa[rt][ks] = 0.f;
          if (r < K_in && ks < KS)
            fa[rt][ks] = as_global(static_cast<const float*>(v.state_in))[((int64_t)b * K_in + r) * e +
                                                                         ks * 4 + g];
        }
      }
      float w[KST], a0;
      auto load_w = [&](int ct) {
        const int t = ct < n_ct ? ct : n_ct - 1;
        a0 = as_global(Arow)[t * 16 + c];
        const float* p = static_cast<const float*>(v.Wbeam) + t * 16 + c;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) w[ks] = ks < KS ? as_global(p)[(int64_t)(ks * 4 + g) * V] : 0.f;
      };
      load_w(wave);
#pragma unroll 1
      for (int ct = wave; ct < n_ct; ct += kBeamWaves) {
        floatx4 z[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) z[rt] = floatx4{a0, a0, a0, a0};
#pragma unroll
        for (int ks = 0; ks < KST; ++ks)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            z[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[rt][ks], w[ks], z[rt], 0, 0, 0);
        load_w(ct + kBeamWaves);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 16 * rt + 4 * g + i;
            if (r < K_in) zt[r * Vp + ct * 16 + c] = z[rt][i];
          }
      }
    } else {
      // no state: every beam's logits are the user part
      for (int q = tid; q < K_in * (V >> 2); q += kBeamThreads) {
        const int r = q / (V >> 2), col = 4 * (q - r * (V >> 2));
        const uint4 x = load_global_u4(Arow + col);
        *reinterpret_cast<uint4*>(zt + r * Vp + col) = x;
      }
    }
    if (tid == 0) {
      s.n_list = 0;
      s.n_valid = 0;
    }
    __syncthreads();

    // ---- 2. rows ----
    const int q_end = (V + 255) >> 8;                      // a lane's groups of four codes: 256 j + 4 lane
    auto quad = [&](int r, int j) {
      const int col = 256 * j + 4 * lane;
      float4 x = float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      if (col < V) x = *reinterpret_cast<const float4*>(zt + r * Vp + col);
      return x;
    };
    constexpr int RU = RT == 1 ? 2 : 4;                    // beams of a wave side by side
    const uint64_t* const keys = s.key[cur];
    float top = -INFINITY;                                 // this lane's best score
    auto push = [&](float score, int r, int col, unsigned long long at_least) {
      const uint64_t en = beam_entry(score, r, (uint32_t)col);
      if (en >= at_least) {
        const int at = atomicAdd(&s.n_list, 1);
        if (at < a.list_cap) list[at] = en;
      }
    };
#pragma unroll 1
    for (int r0 = wave; r0 < K_in; r0 += kBeamWaves * RU) {
      int row[RU];
      float m[RU], mine[RU], sum[RU], lse[RU], sp[RU];
      uint64_t bits[RU];                                   // prefilter bits of the lane's first codes
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        row[u] = r0 + kBeamWaves * u < K_in ? r0 + kBeamWaves * u : r0;
        m[u] = -INFINITY;
        sum[u] = 0.f;
        sp[u] = s.sp[cur][row[u]];
        if (verify) bits[u] = filter_bits(v.set, keys[row[u]], 4 * lane);
      }
#pragma unroll 1
      for (int j = 0; j < q_end; ++j)
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const float4 x = quad(row[u], j);
          m[u] = fmaxf(m[u], fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)));
        }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        mine[u] = m[u];
        m[u] = wave_max_f(m[u], lane);
      }
#pragma unroll 1
      for (int j = 0; j < q_end; ++j)
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const float4 x = quad(row[u], j);
          sum[u] += (__builtin_amdgcn_exp2f((x.x - m[u]) * kLog2e) + __builtin_amdgcn_exp2f((x.y - m[u]) * kLog2e)) +
                    (__builtin_amdgcn_exp2f((x.z - m[u]) * kLog2e) + __builtin_amdgcn_exp2f((x.w - m[u]) * kLog2e));
        }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        sum[u] = wave_sum_f(sum[u], lane);
        lse[u] = m[u] + __builtin_amdgcn_logf(sum[u]) * kLn2;
        if (lane == 0) s.lse[row[u]] = lse[u];
        top = fmaxf(top, sp[u] + (mine[u] - lse[u]));      // (-inf for an empty slot)
      }
      if (!verify) continue;
      // ---- 5a. the beams' K best codes that can be items ----
      // K-th largest logit: t is raised bit by bit while at least K logits stay at or above it; the
      // K-th largest of the lanes' maxima (a lower bound) and the largest logit share the bits it
      // starts with, and it ends early once exactly K logits are left.
      uint32_t t[RU];
      int held[RU], bit = -1;
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)ordered_bits(m[u]));
        uint32_t lo = K <= 64 ? wave_kth(mine[u] > -INFINITY ? ordered_bits(mine[u]) : 0u, K, 16) : 0u;
        const uint32_t differ = lo ^ hi;
        const int first = differ ? 31 - __builtin_clz(differ) : -1;
        t[u] = first < 0 ? hi : hi & ~((2u << first) - 1u);
        held[u] = -1;
        bit = first > bit ? first : bit;
      }
#pragma unroll 1
      for (; bit >= 0; --bit) {
        int cnt[RU];
        float cand[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          cnt[u] = 0;
          cand[u] = unordered_bits(t[u] | (1u << bit));
        }
#pragma unroll 1
        for (int j = 0; j < q_end; ++j)
#pragma unroll
          for (int u = 0; u < RU; ++u) {
            const float4 x = quad(row[u], j);
            cnt[u] += __popcll(__ballot(x.x >= cand[u])) + __popcll(__ballot(x.y >= cand[u])) +
                      __popcll(__ballot(x.z >= cand[u])) + __popcll(__ballot(x.w >= cand[u]));
          }
        bool all = true;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const uint32_t next = t[u] | (1u << bit);
          if (held[u] != K && cnt[u] >= K && next != t[u]) {
            t[u] = next;
            held[u] = cnt[u];
          }
          all = all && held[u] == K;
        }
        if (all) break;
      }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        if (r0 + kBeamWaves * u >= K_in || keys[row[u]] == kEmpty) continue;   // wave uniform
        const float tf = unordered_bits(t[u]);
        int ties = 1 << 30;                                // how many of the logits equal to t are taken
        if (held[u] != K) {
          int above = 0;
          for (int j = 0; j < q_end; ++j) {
            const float4 x = quad(row[u], j);
            above += __popcll(__ballot(x.x > tf)) + __popcll(__ballot(x.y > tf)) +
                     __popcll(__ballot(x.z > tf)) + __popcll(__ballot(x.w > tf));
          }
          ties = K - above;
        }
        int seen = 0;
#pragma unroll 1
        for (int j = 0; j < q_end; ++j) {
          const int col = 256 * j + 4 * lane;
          const uint64_t w = j == 0 ? bits[u] : filter_bits(v.set, keys[row[u]], col);
          const float4 x = quad(row[u], j);
          const float xs[4] = {x.x, x.y, x.z, x.w};
          uint32_t take = 0;
          if (held[u] == K) {
#pragma unroll
            for (int k = 0; k < 4; ++k) take |= (xs[k] >= tf ? 1u : 0u) << k;
          } else {
            // equal to the K-th: the lower codes are taken
            uint64_t eq[4];
            int before = seen;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              eq[k] = __ballot(xs[k] == tf);
              before += lane_rank(eq[k]);
              seen += __popcll(eq[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              take |= (xs[k] > tf || (xs[k] == tf && before < ties) ? 1u : 0u) << k;
              before += xs[k] == tf ? 1 : 0;
            }
          }
          take &= (uint32_t)(w >> (col & 63));
          if (take != 0u && col < V)
#pragma unroll 1
            for (int k = 0; k < 4; ++k)
              if ((take >> k) & 1u)
                push(sp[u] + ((k == 0 ? xs[0] : k == 1 ? xs[1] : k == 2 ? xs[2] : xs[3]) - lse[u]), row[u],
                     col + k, 0ull);
        }
      }
    }
    // A score that at least K of the values given (one per lane of the workgroup) reach, as ordered
    // bits (0: none): the K-th largest of a wave, or the smallest of the waves' q-th largest.
    auto threshold = [&](float best, int waves) {
      const uint32_t x = best > -INFINITY ? ordered_bits(best) : 0u;
      const int q = (K + waves - 1) / waves;
      const uint32_t bk = K <= 64 ? wave_kth(x, K, 18) : 0u;
      const uint32_t bq = q <= 64 ? wave_kth(x, q, 18) : 0u;
      if (lane == 0) {
        s.bound_k[wave] = bk;
        s.bound_q[wave] = wave < waves ? bq : ~0u;
      }
      __syncthreads();
      uint32_t most = 0, least = ~0u;
#pragma unroll
      for (int w = 0; w < kBeamWaves; ++w) {
        most = s.bound_k[w] > most ? s.bound_k[w] : most;
        least = s.bound_q[w] < least ? s.bound_q[w] : least;
      }
      return most > least ? most : least;
    };
    int n;
    if (!verify) {
      // ---- 3. threshold, 4. list ----
      unsigned long long t64 = (unsigned long long)threshold(top, K_in < kBeamWaves ? K_in : kBeamWaves) << 32;
#pragma unroll 1
      for (;;) {
        const float tau = t64 ? unordered_bits((uint32_t)(t64 >> 32)) : -INFINITY;
#pragma unroll 1
        for (int r0 = wave; r0 < K_in; r0 += kBeamWaves * RU) {
          float sp[RU], lse[RU];
#pragma unroll
          for (int u = 0; u < RU; ++u) {
            const int r = r0 + kBeamWaves * u < K_in ? r0 + kBeamWaves * u : r0;
            sp[u] = s.sp[cur][r];
            lse[u] = s.lse[r];
          }
#pragma unroll 1
          for (int j = 0; j < q_end; ++j) {
            float4 x[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
              const int r = r0 + kBeamWaves * u;
              x[u] = quad(r < K_in ? r : r0, j);
            }
            const int col = 256 * j + 4 * lane;
#pragma unroll
            for (int u = 0; u < RU; ++u) {
              const int r = r0 + kBeamWaves * u;
              const float sc[4] = {sp[u] + (x[u].x - lse[u]), sp[u] + (x[u].y - lse[u]),
                                   sp[u] + (x[u].z - lse[u]), sp[u] + (x[u].w - lse[u])};
              if (fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])) >= tau && sp[u] > -INFINITY && col < V &&
                  r < K_in) {
#pragma unroll 1
                for (int k = 0; k < 4; ++k) {
                  const float one = k == 0 ? sc[0] : k == 1 ? sc[1] : k == 2 ? sc[2] : sc[3];
                  if (one >= tau) push(one, r, col + k, t64);
                }
              }
            }
          }
        }
        __syncthreads();
        n = s.n_list;
        if (n <= a.list_cap) break;
        // ties: the K-th best of the first 512 listed is a tighter threshold (512 - K of them go)
        __syncthreads();
        {
          const uint64_t me = list[tid];
          int above = 0;
          for (int j = 0; j < kBeamThreads; ++j) above += list[j] > me;
          if (above == K - 1) s.t64 = me;
        }
        if (tid == 0) s.n_list = 0;
        __syncthreads();
        t64 = s.t64;
      }
    } else {
      // ---- 5b. look the candidates up ----
      __syncthreads();
      n = s.n_list;                                        // at most K_in * K, which fit the list
      constexpr int PER = 8;
      uint32_t ok = 0;
      uint64_t mine[PER];
      float best = -INFINITY;
#pragma unroll 1
      for (int u = 0; u * kBeamThreads < n; ++u) {
        const int i = tid + u * kBeamThreads;
        if (i < n) {
          const uint64_t en = list[i];
          if (set_probe(v.set, keys[entry_parent(en)] + (uint64_t)entry_code(en) * v.set.mult_last)) {
            ok |= 1u << u;
            best = fmaxf(best, entry_score(en));
          }
        }
      }
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int i = tid + u * kBeamThreads;
        mine[u] = i < n ? list[i] : 0ull;
      }
      uint32_t tau_bits = 0;
      if (n > kBeamThreads) tau_bits = threshold(best, kBeamWaves);   // a dense set: not all of them go on
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        if (u * kBeamThreads >= n) break;
        const bool in = ((ok >> u) & 1u) && (uint32_t)(mine[u] >> 32) >= tau_bits;
        const uint64_t bal = __ballot(in);
        if (bal == 0ull) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s.n_valid, __popcll(bal));
        at = __builtin_amdgcn_readfirstlane(at) + lane_rank(bal);
        if (in) list[at] = mine[u];
      }
      __syncthreads();
      n = s.n_valid;
    }
    // ---- 6. places, outputs, Transition ----
    const int nxt = cur ^ 1;
    const int cnt = n < K ? n : K;
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
    cur = nxt;
    if (v.state_out) {
      __syncthreads();
      if (v.transition == NEZHA_TRANSITION_RNN)
        update_states_rnn<false>(v.state_in, v.E, v.U, v.state_out, b, K, K_in, e, s.fin_parent, s.fin_code,
                                 tid, kBeamThreads);
      else
        update_states<false>(v.state_in, v.E, v.state_out, b, K, K_in, e, s.fin_parent, s.fin_code, tid,
                             kBeamThreads);
      __threadfence_block();                               // the next level reads the states back
    }
    __syncthreads();
  }
}
