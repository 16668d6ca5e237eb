// Shapes of a tile's parts (host only; evaluated at compile time by its test).
#pragma once

namespace gs {

// A rectangle of 2^log2_w x 2^log2_h pixels, 2^log2_nx of which lie side by side.
struct Part {
  int log2_w, log2_h, log2_nx;
};

// 2^log2_parts equal parts of a 2^log2_w x 2^log2_h rectangle, as square as it
// allows (wider on ties): a tile's sub-tiles, one per wave, and a sub-tile's
// blocks of 64 pixels.  At least 2^log2_parts pixels.
constexpr Part split(int log2_w, int log2_h, int log2_parts) {
  Part best{-1, -1, -1};
  int dbest = 0;
  for (int nx = 0; nx <= log2_parts; ++nx) {
    const int w = log2_w - nx, h = log2_h - (log2_parts - nx);
    if (w < 0 || h < 0) continue;
    const int d = w > h ? w - h : h - w;
    if (best.log2_nx < 0 || d < dbest || (d == dbest && w > best.log2_w)) {
      best = Part{w, h, nx};
      dbest = d;
    }
  }
  return best;
}

}  // namespace gs
