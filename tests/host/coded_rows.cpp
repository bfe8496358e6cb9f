// Every load of the row kernels that read column codes, walked on the host with
// the kernels' own index functions: for each matrix size, grid and block size,
// the rows each wave takes, the records, values and x it loads.  Exits with the
// number of sizes at which a load is out of range or a row is not taken exactly once.
//   coded_rows FIRST LAST [all-waves]
// all-waves: as if waves past the matrix summed the last slice too.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "amg_index.hpp"

using namespace amg;

namespace {
// The matrix: the diagonal, and entries at +-1, +-d and +-e where both rows exist.
bool entry(int row, int n, int off) { return row + off >= 0 && row + off < n; }

bool sound(int n, int rb, int grid, int d, int e, bool all_waves) {
    const int offs[7] = {-e, -d, -1, 0, 1, d, e};
    const int slices = (n + kWave - 1) / kWave;
    std::vector<int> seen(n, 0);
    for (int block = 0; block < grid; ++block) {
        const BlockRange r = xcd_range((n + rb - 1) / rb, block, grid);
        for (int w = 0; w < rb / kWave; ++w) {
            const int ahead = slice_at(wave_slice(r.first, rb, w), n);
            if (ahead < 0 || ahead >= slices) return false;
            for (int b = r.first; b < r.end; b += r.step) {
                const int own = wave_slice(b, rb, w), next = slice_at(wave_slice(b + r.step, rb, w), n);
                if (next < 0 || next >= slices) return false;
                for (int lane = 0; lane < kWave; ++lane) {
                    const int row = b * rb + w * kWave + lane;
                    if (row < n) ++seen[row];
                }
                if (!wave_has_rows(own, n) && !all_waves) continue;
                const int s = slice_at(own, n);
                int total = 0;
                for (int k = 0; k < 7; ++k)
                    for (int lane = 0; lane < kWave; ++lane) {
                        // the record's bit: the lane's row of slice s has an entry at offs[k]
                        const int at = s * kWave + lane, row = b * rb + w * kWave + lane;
                        const bool on = at < n && entry(at, n, offs[k]);
                        total += on;
                        const int c = coded_col(row, n, on, offs[k]);
                        if (c < 0 || c >= n) return false;
                    }
                for (int k = 0; k < 8 * kWave; ++k) {
                    const int v = coded_val(k, total - 1);
                    if (v < 0 || v >= total) return false;
                }
            }
        }
    }
    for (int c : seen)
        if (c != 1) return false;
    return true;
}
}  // namespace

int main(int argc, char** argv) {
    if (argc < 3) return 255;
    const bool all_waves = argc > 3;
    int bad = 0;
    for (int n = atoi(argv[1]); n <= atoi(argv[2]); ++n)
        for (int rb = 128; rb <= 512; rb *= 2) {
            const int nb = (n + rb - 1) / rb;
            bool ok = true;
            for (int grid : {8, 11, nb})
                if (grid <= nb) ok = ok && sound(n, rb, grid, 2, 64 + n % 7, all_waves);
            if (!ok) {
                if (bad < 10) std::printf("n %d, blocks of %d rows\n", n, rb);
                ++bad;
                break;
            }
        }
    std::printf("%d of the sizes %s to %s are wrong\n", bad, argv[1], argv[2]);
    return bad < 250 ? bad : 250;
}
