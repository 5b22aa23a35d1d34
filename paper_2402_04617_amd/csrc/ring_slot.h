// Slots of the append's rings (position t lies in slot t mod ring), and where it reads the
// keys of the tokens that leave the window.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace infllm {

// Slot of position past + i of the chunk, given slot0 = past mod ring: 0 <= i < n_q < ring,
// so it wraps at most once.
__host__ __device__ inline int ring_slot(int slot0, int i, int ring) {
  return slot0 + i - (slot0 + i >= ring ? ring : 0);
}
// Slot of the token t = pos - n_local that leaves the window at position pos, whose slot is
// sp.  Where t has scores (t >= n_init) the host checked that the ring still holds it, so
// n_local < ring.  A ring may be shorter than the window while no token leaves it (a short
// chunk near the start): the position's own slot then stands in, and its value is not used.
__host__ __device__ inline int leaving_slot(int64_t pos, int n_local, int n_init, int sp, int ring) {
  if (pos - n_local < n_init) return sp;
  return sp - n_local + (sp < n_local ? ring : 0);
}
// Whether the key of token t that leaves the window is read from the chunk (which may be
// absent where the caller stored it before): only where t has scores, which the host then
// checked it is given for.  Any other key comes from the store, its value used or not.
__host__ __device__ inline bool leaving_key_in_chunk(int64_t past, int64_t t, int n_init) {
  return t >= past && t >= n_init;
}

}  // namespace infllm
