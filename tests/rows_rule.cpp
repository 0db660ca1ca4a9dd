// Prints the rows rule's answer for each line "n T elem obs reward" read.
#include <stdio.h>

#include "cp_rows.h"

int main() {
  unsigned n, elem;
  unsigned long long T, obs, reward;
  while (scanf("%u %llu %u %llu %llu", &n, &T, &elem, &obs, &reward) == 5)
    printf("%u\n", cp::rows_block(n, T, elem, uintptr_t(obs), uintptr_t(reward)));
  return 0;
}
