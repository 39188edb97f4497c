// The autotuner's choice from its measurements.
#pragma once

// The index of the smallest of n times (ties: the lower index), or `base`, the variant an
// untuned launch takes, unless that is slower by more than the fraction `margin`.
inline int pick_variant(const double* time, int n, int base, double margin) {
  int v = 0;
  for (int i = 1; i < n; ++i)
    if (time[i] < time[v]) v = i;
  return time[v] < time[base] * (1.0 - margin) ? v : base;
}
