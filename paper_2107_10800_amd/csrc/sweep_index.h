// LDS of the symmetric block sweep (pc_sweep_kernel in precond.hip): where its blocks of
// 16 rows lie and which of them a tile's update reads.  Plain arithmetic, in doubles from
// the start of the dynamic LDS, so that its bounds can be checked without a device.
#pragma once

namespace arb {

constexpr int kSwLd = 17;      // row stride
constexpr int kSwNone = 255;   // tile row and column of a slot without a tile
constexpr int kSwMaxWaves = 8;

// matrices of nb tile rows: two buffers of C_r = A_rk (this and the next step), -W_r, then
// two blocks each (even and odd steps) of P, P^T and A_kk before its update; the
// transposes at the end take a block per wavefront from the start
struct SweepLds {
    int buf, W, P, T, D, end;
};
constexpr SweepLds sweep_lds(int nb) {
    const int block = 16 * kSwLd, buf = nb * block, W = 2 * buf, P = W + buf, T = P + 2 * block,
              D = T + 2 * block, end = D + 2 * block, tr = kSwMaxWaves * block;
    return SweepLds{buf, W, P, T, D, end > tr ? end : tr};
}

// the operands of tile (i, j) in step k, A_ij -= W_i C_j^T (row and column k: see the
// kernel).  A slot without a tile (i = j = kSwNone) runs along with the others of its run
// and reads the last block row
constexpr int sweep_operand_a(const SweepLds &L, int nb, int i) {
    return L.W + 16 * (i < nb ? i : nb - 1) * kSwLd;
}
constexpr int sweep_operand_b(const SweepLds &L, int nb, int i, int j, int k) {
    const int r = 16 * (j < nb ? j : nb - 1) * kSwLd;
    return i != k ? (k & 1) * L.buf + r : (j != k ? L.W + r : L.T + 16 * (k & 1) * kSwLd);
}

}  // namespace arb
