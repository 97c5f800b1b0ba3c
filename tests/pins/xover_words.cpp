// Host build of the crossover draws that share rounds between rows and
// columns (XoverCol, XoverRow), against the same block drawn whole.
// One query per line: run gen indiv q key_lo key_hi; one answer per line:
// the four words drawn with shared rounds, then the four of draw_block.
#include <cstdio>

#include "de_device.hpp"

int main() {
  unsigned run, gen, i, q, k0, k1;
  while (std::scanf("%u %u %u %u %u %u", &run, &gen, &i, &q, &k0, &k1) == 6) {
    const de::Words4 a =
        de::xover_words(de::xover_col(run, gen, q, k0, k1),
                        de::xover_row(gen, i, k0, k1), k0, k1);
    const de::Words4 b =
        de::draw_block(de::kTagXover, run, gen, i, q, k0, k1);
    std::printf("%u %u %u %u %u %u %u %u\n", a.w[0], a.w[1], a.w[2], a.w[3],
                b.w[0], b.w[1], b.w[2], b.w[3]);
  }
  return 0;
}
