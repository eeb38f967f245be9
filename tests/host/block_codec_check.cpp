// Host-only driver for the per-block coder and decoder (for sanitizer runs).
//   block_codec_check enc|dec RATE KERNEL_RATE VAR MAXPREC MINEXP COUNT
// reads COUNT blocks (enc: 64 floats each, dec: RATE 64-bit words each) from
// stdin and writes what they code or decode to (enc: RATE words, then all the
// lengths in bits; dec: 64 floats).  KERNEL_RATE is the rate the code is built
// for (0: any).  Every slice is a heap allocation of just the words that a lane
// has on the device, so that an access outside it is reported.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <memory>
#include <vector>

#include "../../paper_2609_24294_amd/csrc/block_codec.hpp"

using namespace zfpx;

template <int RATE, bool VAR>
static void encode(const float* in, int n, int rate, int maxprec, int minexp, uint64_t* out,
                   uint32_t* bits) {
  for (int b = 0; b < n; b++) {
    float v[64];
    memcpy(v, in + 64 * (size_t)b, sizeof v);
    std::unique_ptr<uint64_t[]> slice(new uint64_t[rate + kSlackWords]());
    bits[b] = encode_block<RATE, VAR>(v, slice.get(), rate, maxprec, minexp);
    memcpy(out + (size_t)b * rate, slice.get(), 8 * (size_t)rate);
  }
}

template <int RATE, bool VAR>
static void decode(const uint64_t* in, int n, int rate, int maxprec, int minexp, float* out) {
  for (int b = 0; b < n; b++) {
    std::unique_ptr<uint64_t[]> slice(new uint64_t[rate + kSlackWords]());
    memcpy(slice.get(), in + (size_t)b * rate, 8 * (size_t)rate);
    decode_block<RATE, VAR>(slice.get(), out + 64 * (size_t)b, rate, maxprec, minexp);
  }
}

template <int RATE, bool VAR>
static int run(bool enc, int rate, int maxprec, int minexp, int n) {
  std::vector<float> f(64 * (size_t)n);
  std::vector<uint64_t> w((size_t)rate * n);
  std::vector<uint32_t> bits(n);
  if (enc) {
    if (fread(f.data(), 256, n, stdin) != (size_t)n) return 2;
    encode<RATE, VAR>(f.data(), n, rate, maxprec, minexp, w.data(), bits.data());
    fwrite(w.data(), 8, w.size(), stdout);
    fwrite(bits.data(), 4, n, stdout);
  } else {
    if (fread(w.data(), 8, w.size(), stdin) != w.size()) return 2;
    decode<RATE, VAR>(w.data(), n, rate, maxprec, minexp, f.data());
    fwrite(f.data(), 4, f.size(), stdout);
  }
  return 0;
}

template <int RATE>
static int run(bool var, bool enc, int rate, int maxprec, int minexp, int n) {
  if (RATE > 0 && rate != RATE) return 2;
  return var ? run<RATE, true>(enc, rate, maxprec, minexp, n)
             : run<RATE, false>(enc, rate, maxprec, minexp, n);
}

int main(int argc, char** argv) {
  if (argc != 8) return 2;
  const bool enc = strcmp(argv[1], "enc") == 0, var = atoi(argv[4]) != 0;
  const int rate = atoi(argv[2]), mp = atoi(argv[5]), me = atoi(argv[6]), n = atoi(argv[7]);
  if (rate < 1 || rate > 32 || n < 1) return 2;
  switch (atoi(argv[3])) {
    case 0: return run<0>(var, enc, rate, mp, me, n);
    case 8: return run<8>(var, enc, rate, mp, me, n);
    case 16: return run<16>(var, enc, rate, mp, me, n);
    case 32: return run<32>(var, enc, rate, mp, me, n);
    default: return 2;
  }
}
