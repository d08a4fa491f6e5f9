// LDS of one workgroup of the Newton and adjoint kernels.
#pragma once

namespace pfx {

struct NrLayout {
  int xs, tmp, red, redn, H, cs, sn, gres, gfin, y, w, total;
};

constexpr int align16(int x) { return (x + 15) & ~15; }

// Column j of the packed Hessenberg matrix holds rows 0..j at offset j(j+1)/2.
constexpr int hcol(int j) { return j * (j + 1) / 2; }

// Entries of `ts` bytes of the dense core's right-hand side: k and the zeros up
// to four parts of whole 16-byte packs.
constexpr int core_entries(int k, int ts) {
  const int P = 16 / ts;
  return ((k + P - 1) / P + 3) / 4 * 4 * P;
}

constexpr NrLayout nr_layout(int nbp, int nth, int npq, int kmax, int R, int NW, bool split, int ts) {
  NrLayout L{};
  int o = 0;
  int xs_bytes = 2 * nbp * 8;                          // V (FP64 pairs) in the mismatch
  if (2 * nbp * ts > xs_bytes) xs_bytes = 2 * nbp * ts;  // dV pairs in the Jacobian-vector product
  // the preconditioner's two right-hand sides and pass buffers: [0, 2 nth) and [nth, nth + npq)
  if (2 * nth * ts > xs_bytes) xs_bytes = 2 * nth * ts;
  if ((nth + npq) * ts > xs_bytes) xs_bytes = (nth + npq) * ts;
  L.xs = o;
  o += align16(xs_bytes);
  // Reduction partials, double-buffered.  The preconditioner's dense-core
  // right-hand side lives there too when it fits: no partial is pending while
  // the preconditioner runs (each phase in between ends with a barrier).
  const int red_bytes = 2 * (R + 2) * NW * 8;
  L.red = o;  o += align16(red_bytes);
  const int core = (kmax + 3) / 4 * 4 * ts;
  if (core <= red_bytes) {
    L.tmp = L.red;
  } else {
    L.tmp = o;
    o += align16(core);
  }
  // The norm reduction after the projection.  The last zeros of the core's
  // right-hand side may lie over it (a barrier apart, as for the partials), so
  // that they take no LDS of their own: at 8192 buses every byte counts.
  const int zeros = core_entries(kmax, ts) * ts - core;
  L.redn = o; o += align16(zeros > NW * 8 ? zeros : NW * 8);
  L.H = o;    o += align16(hcol(R) * ts);
  L.cs = o;   o += align16(R * ts);
  L.sn = o;   o += align16(R * ts);
  L.gres = o; o += align16((R + 1) * ts);
  L.gfin = o; o += align16(R * ts);
  L.y = o;    o += align16(R * ts);
  L.w = o;    // a split FP32 workgroup's vector for its sums
  if (split && ts == 4) o += align16(2 * nbp * ts);
  L.total = o;
  return L;
}

}  // namespace pfx
