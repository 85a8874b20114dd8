// Prints the shape of a dock launch (lanes per orientation, waves, parts, two waves a chunk) for each line
// of its input: ligands, atoms, largest ligand, most bonds, the sums over the ligands of n^2, moving atoms and
// (moving, fixed) pairs of their bonds and of the bonds, orientations, turns, passes, offsets, top_k, compute units.
#include <cstdio>

#include "exs_internal.h"

int main() {
    int n, n_max, rot_max, K, S, P, T, top_k, cus;
    double atoms, square, moving, pairs, bonds;
    while (std::scanf("%d %lf %d %d %lf %lf %lf %lf %d %d %d %d %d %d", &n, &atoms, &n_max, &rot_max, &square, &moving, &pairs,
                      &bonds, &K, &S, &P, &T, &top_k, &cus) == 14) {
        exs::WorkSums sums;
        sums.ligands = n;
        sums.atoms = atoms;
        sums.square = square;
        sums.moving = moving;
        sums.pairs = pairs;
        sums.bonds = bonds;
        exs::LaunchWork w = sums.mean(S, P, T);
        w.n_lig = n;
        w.n_atoms = (int64_t)atoms;
        w.n_max = n_max;
        w.rot_max = rot_max;
        const exs::DockShape sh = exs::dock_shape(w, K, S, top_k, cus);
        std::printf("%d %d %d %d\n", sh.lanes, sh.waves, sh.parts, sh.pair ? 1 : 0);
    }
    return 0;
}
