// TTPairWalk (tt_internal.h): every chunk of a walk against the pairs counted one by one, and the ends of walks of 2^31
// pairs and more, where a 32-bit pair number would overflow.  Prints "ok" or the first difference.
#include <stdio.h>
#include "tt_internal.h"

static bool check(int nq, int d) {  // all pairs in order
  unsigned mul, sh;
  tt_div_constants(d, &mul, &sh);
  TTPairWalk<64> w(nq, d, mul, sh);
  int s = 0, j = 0;
  for (int n; (n = w.count()) > 0; w.advance())
    for (int k = 0; k < n; ++k) {
      int ps, pj;
      w.pair(k, ps, pj);
      if (ps != s || pj != j) { printf("nq %d d %d: pair (%d, %d) instead of (%d, %d)\n", nq, d, ps, pj, s, j); return false; }
      if (++j == d) { j = 0; ++s; }
    }
  w.advance();
  if (s != nq || j != 0 || w.count() != 0) { printf("nq %d d %d: ended at (%d, %d)\n", nq, d, s, j); return false; }
  return true;
}

static bool check_long(int nq, int d) {  // the chunks' sizes add up, the last pair is the last one
  unsigned mul, sh;
  tt_div_constants(d, &mul, &sh);
  TTPairWalk<64> w(nq, d, mul, sh);
  long long sum = 0;
  int ps = -1, pj = -1;
  for (int n; (n = w.count()) > 0; w.advance()) { sum += n; w.pair(n - 1, ps, pj); }
  if (sum != (long long)nq * d || ps != nq - 1 || pj != d - 1) { printf("nq %d d %d: %lld pairs, last (%d, %d)\n", nq, d, sum, ps, pj); return false; }
  return true;
}

int main() {
  const int ds[] = {1, 2, 3, 4, 5, 7, 31, 32, 63, 64, 65, 100, 127, 128, 1000, 1023, 1024}, nqs[] = {0, 1, 2, 15, 16, 17, 63, 64, 65, 200};
  for (int d : ds)
    for (int nq : nqs)
      if (!check(nq, d)) return 1;
  if (!check_long(2100000, 1023) || !check_long(2097152, 1024) || !check_long(2147483646, 1) || !check_long(2147483646, 2)) return 1;
  printf("ok\n");
  return 0;
}
