#pragma once
#include <cstdint>

// A workgroup of 256 threads for each of N = 2^L proofs.  A launch dimension takes fewer than 2^32
// threads, which N workgroups reach at L = 24 (203 GB of proofs at b = 1 fit the device), so that
// more than 2^16 of them spread over two dimensions: proof blockIdx.y 2^16 + blockIdx.x.
struct ProofGrid {
  uint32_t x, y;
};
constexpr ProofGrid proof_grid(uint64_t N) {
  return N <= 65536 ? ProofGrid{(uint32_t)N, 1} : ProofGrid{65536, (uint32_t)(N >> 16)};
}
