// Host-only helpers shared by the C ABI implementation and the packer.
#pragma once
#include <stdint.h>

#include "../../include/sph.h"

int sph_host_check_format(const sph_format* fmt);
int sph_host_check_shape(int64_t n, int64_t k);
int sph_host_layout(const sph_format* fmt, int64_t n, int64_t k, uint64_t off[8], uint64_t* total);
int sph_host_check_codes(const sph_format* fmt, int64_t n, int64_t k, const uint8_t* signs,
                         const uint16_t* dir_idx, const uint8_t* radius_code, const uint16_t* gmin,
                         const uint16_t* gstep, const uint16_t* codebook);
void sph_host_pack(const sph_format* fmt, int64_t n, int64_t k, const uint8_t* signs,
                   const uint16_t* dir_idx, const uint8_t* radius_code, const uint16_t* gmin,
                   const uint16_t* gstep, const uint16_t* codebook, const uint64_t off[8],
                   uint8_t* blob);

// Whether every weight's radius times direction fits two fp16 words at the precision of an fp32
// product (SPH_FLAG_RADIUS_SPLIT): codes already checked by sph_host_check_codes.
bool sph_host_radius_split(const sph_format* fmt, int64_t n, int64_t k, const uint16_t* gmin, const uint16_t* gstep,
                           const uint16_t* codebook);

// Workgroups of the encoder's small-codebook kernel: 4 waves of 256 threads take 64 vectors each and go on in steps
// of the grid, which stays below the 2^32 threads that a launch may have (a matrix may have 2^35 vectors).
constexpr int kEncodeWaves = 4;

static inline unsigned sph_encode_blocks(int64_t units) {
  const int64_t b = (units + kEncodeWaves - 1) / kEncodeWaves;
  return (unsigned)(b < (int64_t(1) << 22) ? b : int64_t(1) << 22);
}
