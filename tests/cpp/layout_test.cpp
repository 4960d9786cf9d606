// Host-side rules that the kernels share with the layout header.
#include <stdint.h>
#include <stdio.h>

#include "../../paper_2201_13020_amd/csrc/szx_layout.hpp"

#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
      return 1;                                               \
    }                                                         \
  } while (0)

int main() {
  // the encoder reads no entry of a list that a failed classification may have
  // left with gaps
  CHECK(szx::listed_tiles(0, 191) == 191);
  CHECK(szx::listed_tiles(0, 0) == 0);
  CHECK(szx::listed_tiles(1, 191) == 0);
  CHECK(szx::listed_tiles(0x80000000u, ~0ull) == 0);

  // a launch beside the encode pass may hold the device for seconds before the
  // pass's later workgroups start: the scan workgroup outlasts that, and a
  // tile's wait, which is for running workgroups, stays short (0.19 us a poll)
  CHECK(0.19e-6 * szx::kScanSpinLimit >= 10.0);
  CHECK(0.19e-6 * szx::kSpinLimit < 0.1);

  // the encode workgroups of a launch and its two scan workgroups fit the device
  // at once (160 KiB of LDS a compute unit; a workgroup's rings take its tile)
  for (uint32_t w : {4u, 8u})
    for (uint32_t b : {8u, 16u, 32u, 64u, 128u, 256u, 512u, 1024u}) {
      const uint32_t tile = szx::enc_blocks(b, w) * b * w;
      for (uint32_t cus : {1u, 64u, 256u}) {
        const uint32_t n = szx::default_encode_wgs(cus, b, w) + 2;
        CHECK(n <= cus * ((160u << 10) / (tile + 1024u)) && n <= cus * 4);
        CHECK(n >= cus * 2);
      }
    }

  printf("layout ok\n");
  return 0;
}
