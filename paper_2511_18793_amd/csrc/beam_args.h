// Arguments of the kernel that runs the levels of a decode for beams of up to 128 (beam_level.h), and
// the launchers of its instances (beam.hip, compiled once per width of the state).
#pragma once
#include "nezha_internal.h"

namespace nezha {

struct BeamLevel {
  const void* state_in;     // [B, K_in, e] or NULL (zero); used unless the states are carried in LDS
  const void* Wbeam;        // bf16: packed beam part of W_l; float32: rows d.. of W_l, row major
  const float* A;           // [B, T_l] user part
  const uint64_t* key_in;   // [B, K_in] or NULL
  const float* score_in;    // [B, K_in] or NULL
  const void* E;            // [T_l, e] (used when state_out != NULL)
  const void* U;            // [e, e] row major (recurrent Transition), else unused
  SetView set;              // slots == NULL: no set is consulted at this level
  uint64_t mult;            // prod_{j<level} T_j
  uint64_t* key_out;
  float* score_out;
  int32_t* parent_out;
  int32_t* code_out;
  void* state_out;          // or NULL
  int32_t* count_out;       // or NULL
  int K_in, V, transition;
};
struct BeamArgs {
  BeamLevel lv[NEZHA_MAX_LEVELS];
  int L, K, e;
  int list_cap;             // entries of the candidate list in LDS (a multiple of 512)
  int state_bufs;           // 0: states pass through global memory only; 1, 2: LDS copies
  int mask_in_lds;          // the set's prefilter bits of a level fit region x
  uint32_t x_off, list_off, state_off, status_off;   // byte offsets in dynamic LDS
};

// (beam_level.h has the kernel)
constexpr int kBeamWaves = 8, kBeamThreads = 64 * kBeamWaves;
constexpr int kBeamList = 2048;            // candidates a level lists in LDS (beam_kernel)
constexpr int kBeamStatusBytes = 2 * (kBeamList + 256);   // their states, and which of them are open
constexpr int kBeamMax = NEZHA_MAX_BEAM;

// One launcher per translation unit: KST matrix steps over the state (bf16: e <= 32 KST; float32:
// e <= 4 KST).  row_tiles = ceil(K / 16); lds: bytes of dynamic LDS.
int launch_beam_1(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);
int launch_beam_2(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);
int launch_beam_3(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);
int launch_beam_4(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);
int launch_beam_8(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);

int launch_decode_lds_16(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);
int launch_decode_lds_32(const BeamArgs& a, int B, int row_tiles, size_t lds, hipStream_t stream);

// Bytes of LDS that do not depend on the shape (BeamShared, DecodeShared).
size_t beam_shared_bytes();
size_t decode_shared_bytes();

}  // namespace nezha
