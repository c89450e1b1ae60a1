// Sample numbers of a trace run up to 2^31 - 3: arithmetic on them that could
// leave 32 bits, in a form that cannot.  (No device code: also tested on the host.)
#pragma once

namespace e2e {

// Sample number, not a whole one, of the place tau in [-1, 1] between the first
// (ks) and the last (ke - 1) sample of a column.
__host__ __device__ inline double node_sample(int ks, int ke, double tau)
{
    return 0.5 * __builtin_fma((double)(ke - 1 - ks), tau, (double)ks + (double)(ke - 1));
}

}  // namespace e2e
