/* How many tiles of 64 positions a wave of the score kernel takes (plain C: the same text is compiled into the library and
 * into a host test).
 *
 * One while all workgroups are resident at once (their LDS decides), two beyond if that saves a round: a second round pays
 * its block sums and first-tile latency again, so a second one of a few workgroups costs what one tile each would.  Four in
 * large calls that score a tile for four or more query heads (8192 positions x 24 sequences: two cost 10 % there, four
 * cost one-head calls 3 %).
 * Selection in two launches, us, one tile / two: two tiles make it one round, 32 heads x 128, three sequences of 2213
 * 19.0 / 17.0, nine of 250 to 525 (40 heads) 16.8 / 15.7, one of 8000 22.7 / 21.1; 16 heads x 64, twelve of 1298 to 2806 17.7 / 16.5;
 * they leave a second round that is nearly empty, 16 heads x 128, seventeen of 515 to 567 17.6 / 19.4, 32 heads, ten of 853 20.7 /
 * 21.9, seven of 627 to 1310 18.8 / 19.9, 8 KV heads, thirteen of 2108 to 2710 25.1 / 26.7 (with lengths that happen to fit one
 * round it is the other way round, 32 heads, thirteen of 244 to 743 21.0 / 18.6, but they are on the device); more than that
 * 32 heads, eleven of 1350 30.5 / 30.0, 40 heads, seven of 1143 to 1287 27.8 / 25.5; all resident, one of 1024 8.4 / 9.8, 8 KV heads,
 * seven of 1811 to 2517 15.5 / 18.6.  Lists of little more than 256 fill two tiles badly: 40 heads, 25 of 67 to 516 28.4 / 30.1.
 * Over 1000 batches the choice is 0.75 % above the better one in the mean (one tile while all are resident and two beyond:
 * 0.9 %; two from 2048 workgroups of one tile on: 3.3 %).  Lists of a little less than three times 256, which two tiles serve
 * in two workgroups instead of three, are left at one although two win there: 32 heads, sixteen of 674 to 782 30.6 / 27.0.
 */
#ifndef DLLM_SCORE_RULES_H
#define DLLM_SCORE_RULES_H
#include <stdint.h>

/* row_bytes: of one K row of one head */
static inline int dllm_rule_score_tiles(int32_t batch, int32_t total_kv, int32_t max_kv, int32_t hkv, int32_t group, int32_t row_bytes) {
  const int rows = 256;   /* positions of a workgroup of four waves with one tile each */
  const double resident = 256.0 * (160 * 1024 / (rows * row_bytes + 4096));
  const double tiles = (double)total_kv * hkv / rows;
  if (group >= 4 && tiles >= 5 * 1024) return 4;
  if (tiles <= resident) return 1;
  /* Workgroups with one and with two tiles per wave: the lengths, which are on the device, are taken to be spread evenly
   * around the mean. */
  double n[2];
  const int reps = batch < 64 ? batch : 64;
  const double mean = (double)total_kv / batch;
  for (int t = 1; t <= 2; ++t) {
    double sum = 0.0;
    for (int i = 0; i < reps; ++i) {
      const double length = max_kv - (max_kv - mean) * (reps > 1 ? 2.0 * i / (reps - 1) : 0.0);
      const int64_t full = length > 0.0 ? (int64_t)(length / (rows * t)) : 0;
      sum += full == 0 || (double)full * (rows * t) < length ? full + 1.0 : (double)full;
    }
    n[t - 1] = sum * batch / reps * hkv;
  }
  return n[1] <= resident || (n[1] > 1.25 * resident && n[1] <= 0.63 * n[0]) ? 2 : 1;
}

#endif
