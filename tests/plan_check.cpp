// Host check of the sizes that scratch memory is planned by: the sort of any
// number of elements up to a capacity stays inside the scratch of that capacity,
// and the loss's one row set inside the workspace that its calls ask for.
#include <cstdio>
#include <vector>

#include "smki_loss_layout.h"

static int bad = 0;
#define CHECK(ok, ...)                 \
  do {                                 \
    if (!(ok) && ++bad < 20) {         \
      printf("wrong: " __VA_ARGS__);   \
      printf("\n");                    \
    }                                  \
  } while (0)

int main() {
  // every count up to 2^20 + 2^13, then around multiples of a tile and powers of two
  std::vector<int64_t> ns;
  for (int64_t n = 1; n <= (1 << 20) + (1 << 13); ++n) ns.push_back(n);
  for (int s = 20; s <= 30; ++s)
    for (int64_t d : {-4097, -4096, -1, 0, 1, 4095, 4096}) {
      const int64_t n = (int64_t(1) << s) + d;
      if (n > ns.back()) ns.push_back(n);
    }
  size_t most = 0;   // written by the sort of some count so far
  for (int64_t n : ns) {
    most = std::max(most, radix_used_bytes(n));
    CHECK(most <= radix_tmp_bytes(n), "capacity %lld: %zu bytes, a smaller sort writes %zu",
          (long long)n, radix_tmp_bytes(n), most);
  }
  printf("radix scratch: %zu counts\n", ns.size());

  // the loss sorts the training rows alone, or rows and queries: both inside the
  // scratch it carves, and the carved set inside what the calls ask for
  const int64_t rows[] = {0,       1,       2,       63,      1000,    4095,    65'536,  65'537,
                          200'000, 250'000, 262'143, 262'144, 262'145, 524'288, 1'048'576,
                          1'048'577, 3'200'000, int64_t(1) << 26, int64_t(1) << 30};
  long cases = 0;
  for (int64_t nt : rows)
    for (int64_t nq : rows)
      for (int32_t K : {2, 20, 64, 65, 255})
        for (int64_t nb : {int64_t(1), int64_t(27), int64_t(30'000), kMaxLossBlocks}) {
          if (nq < 1) continue;
          LossBufs b{};
          const size_t used = carve_body(nullptr, b, nt, nq, K, nb, false);
          ++cases;
          for (int64_t n : {nt, nt + nq})
            CHECK(n < 1 || radix_used_bytes(n) <= b.scr.sort_tmp_bytes,
                  "loss rows %lld queries %lld: a sort of %lld writes %zu of %zu bytes", (long long)nt,
                  (long long)nq, (long long)n, radix_used_bytes(n), b.scr.sort_tmp_bytes);
          CHECK(used <= body_bytes(nt, nq, K, nb), "loss rows %lld queries %lld K %d blocks %lld: %zu > %zu",
                (long long)nt, (long long)nq, K, (long long)nb, used, body_bytes(nt, nq, K, nb));
        }
  printf("loss layout: %ld cases\n", cases);
  // a launch stays below 2^32 threads for as many queries as a call accepts, and
  // starts eight threads for each of few
  for (int64_t nq = 1; nq <= INT32_MAX / 2; nq = nq * 2 - (nq > 1000 ? 1 : 0)) {
    const int64_t threads = 256 * (int64_t)near_mark_grid(nq);
    CHECK(threads < (int64_t(1) << 32), "%lld queries: %lld threads", (long long)nq, (long long)threads);
    CHECK(threads >= std::min<int64_t>(8 * nq, 1 << 21), "%lld queries: %lld threads", (long long)nq,
          (long long)threads);
  }
  printf("near marks\n");
  // rows per unit: whole batches of 64 between 128 and 512, more rows never shorter
  // units nor more slots (from two on) longer ones, and below 512 a unit never more than
  // 4,096 full units (a replay's tables have room for that many beyond its sizing insert's)
  for (int32_t B : {2, 8, 16})
    for (bool few : {false, true})
      for (int64_t slots : {0, 1, 20, 300, 5000, 1'000'000}) {
        const int32_t share = unit_share(B, few);
        int32_t last = 0;
        for (int64_t n = 1; n <= 3'000'000; n += n % 7 + 1) {
          const int32_t c = rows_per_unit(0, share, n, slots);
          CHECK(c % SMKI_WAVE == 0 && c >= 128 && c <= SMKI_CHUNK && c >= last, "%lld rows: %d a unit",
                (long long)n, c);
          CHECK(slots / 2 < 2 || c <= rows_per_unit(0, share, n, slots / 2), "%lld slots", (long long)slots);
          CHECK(c == SMKI_CHUNK || n <= (int64_t)kMostUnits * c, "%lld rows: %d a unit", (long long)n, c);
          last = c;
        }
        CHECK(last == SMKI_CHUNK && rows_per_unit(0, share, INT32_MAX, INT32_MAX) == SMKI_CHUNK &&
                  rows_per_unit(77, share, 5, 5) == 77, "rows per unit");
      }
  // the steps counted for a slot are those of its units, one by one
  for (int32_t rows = 0; rows < 1300; ++rows)
    for (int32_t chunk : {1, 7, 16, 17, 64, 100, 128, 512, 2000}) {
      int64_t want = 0;
      for (int32_t r = 0; r < rows; r += chunk) {
        const int32_t u = std::min(chunk, rows - r);
        want += u <= kFewRows ? u : 33 * ((u + 63) / 64);
      }
      CHECK(lane_steps(rows, chunk, 33) == want, "%d rows, %d a unit: %lld steps", rows, chunk,
            (long long)lane_steps(rows, chunk, 33));
    }
  printf("unit sizes\n");
  if (bad) return printf("%d wrong\n", bad), 1;
  printf("ok\n");
  return 0;
}
