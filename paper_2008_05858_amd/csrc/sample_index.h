// Sample numbers of a trace run up to 2^31 - 3: arithmetic on them that could
// leave 32 bits, in a form that cannot.  (No device code: also tested on the host.)
#pragma once

namespace e2e {

// Sample number, not a whole one, of the place tau in [-1, 1] between the first
// (ks) and the last (ke - 1) sample of a column.
__host__ __device__ inline double node_sample(int ks, int ke, double tau)
{
    return 0.5 * __builtin_fma((double)(ke - 1 - ks), tau, (double)((unsigned)ks + (unsigned)(ke - 1)));
}

// A wave of the table path reads every column's samples as far ahead as its
// longest column goes, so also past the spectrum's end, by up to n of its n
// samples.  A place is therefore kept as its room, the samples between it and
// the spectrum's last g; the g values `off` (0 .. n - 1) past it lie inside if
// off <= room.  (In terms of the index the test wraps above 2^31.  Unsigned
// indices don't, but took 1.17 ms where this takes 1.05 for a 9216^2 frame.)
__host__ __device__ inline int group_room(int n, int g, int place) { return n - g - place; }
__host__ __device__ inline bool group_inside(int room, int off) { return off <= room; }
// Value e of a group that reaches past the end.
__host__ __device__ inline bool value_inside(int room, int g, int off, int e)
{
    return off <= room + (g - 1) - e;
}

}  // namespace e2e
