// Host-side check of the partition's geometry (particles.h), built and run by
// tests/test_host_partition.py: for every mesh and particle count the buckets
// are whole runs of the mesh's keys (64 a tile), no more than the threads of a
// workgroup that counts them, and the counts of a bucket's keys fit 64 KB; and
// what counts as too large a bucket.
#include <cstdio>

#include "particles.h"

int main() {
  using namespace pmk;
  int fails = 0;
  for (int n = 8; n <= 1024; n *= 2) {
    const int t = n / 2 < (n <= 64 ? 8 : 16) ? n / 2 : (n <= 64 ? 8 : 16), side = n / t, ntiles = side * side * side;
    for (long np = kPartitionMin; np < (1L << 31); np += np / 3 + 1) {
      const PartitionGeom p = partition_geom(np, ntiles);
      const bool ok = p.buckets >= 1 && p.buckets <= p.threads && p.threads <= kPartitionBuckets && p.kbits >= 6 &&
                      ((long)p.buckets << p.kbits) == 64L * ntiles && ((size_t)4 << p.kbits) <= 65536;
      if (!ok && ++fails < 20)
        std::printf("FAIL n %d np %ld: %d buckets of 2^%d keys, %d threads\n", n, np, p.buckets, p.kbits, p.threads);
      // a uniform set is not lopsided (its buckets hold the mean, and a few
      // roots of it more), a bucket of half the set is
      const long mean = np / p.buckets;
      if (p.buckets >= 64 && (partition_large(np, p.buckets) < 4 * mean || partition_large(np, p.buckets) > np / 2) &&
          ++fails < 20)
        std::printf("FAIL n %d np %ld: %u is large, the mean %ld\n", n, np, partition_large(np, p.buckets), mean);
    }
  }
  if (fails) return 1;
  std::printf("partition geometry ok\n");
  return 0;
}
