// How the workgroups behind one L2 share the output tiles of a launch whose products differ in depth
// (ns_gemm.hip).
// Plain arithmetic, the same in every workgroup; it also compiles for the host.
#pragma once

namespace mlc {

// A workgroup's share of a product's tiles: at, at + step, ... below end, then at2, at2 + step2, ...
// below end2.
struct Deal { int at, end, step, at2, end2, step2; };

// Products come deepest first, and each is dealt out round by round.  Of the W workgroups the first
// W - late (by `pos`, a permutation of 0 .. W - 1) are about level, and the others are `gap` ahead of
// them: they have more work already.  Work is counted in K tiles, an epilogue as about three, and a triangle
// as a whole tile, though it takes 0.7 to 0.9 of one: who meets more triangles ends sooner than counted here.  So that, in
// this count, no workgroup ends up with more than one deep tile over the average, the level ones first take as many
// whole rounds of a product as fill the gap, and the rest is dealt to all, starting with whoever then
// has less.  Over 7000 drawn sets the longest share is 1.0003 of what dealing each tile to whoever has
// least gives.  (The inner step of 11 x 1280 x 2048 and 20 x 768 x 2816: 1582 us.  With a rule that forgot the
// gap, and began what was left over with those that had just filled it, 1634, and 1 % less than that in
// launches apart.)
struct Dealer { int W, pos, late, gap; };

// `more`: another product follows (the divisions that say how it finds the workgroups take some 0.3 us).
__host__ __device__ __forceinline__ Deal deal_tiles(Dealer& d, int lo, int n, int cost, bool more) {
  const int level = d.W - d.late;
  const int rounds = n && d.late ? (int)((unsigned)(2 * d.gap + cost) / (unsigned)(2 * cost)) : 0;
  const int ahead = rounds * level;
  if (n < ahead) {                   // the level ones take it whole
    const Deal t{d.pos < level ? lo + d.pos : lo + n, lo + n, level, lo + n, lo + n, d.W};
    if (more) {
      const int full = (int)((unsigned)n / (unsigned)level), rest = n - full * level;
      d.gap -= full * cost;
      // those that took one more are now among the late ones, in front of them or behind: whoever has
      // less comes first
      const int among = d.gap > cost ? level : d.W;
      if (d.pos < among) {
        d.pos -= rest;
        if (d.pos < 0) d.pos += among;
      }
      if (rest) {                    // (ahead by the mean of both)
        d.gap = (int)((unsigned)(d.late * d.gap + rest * cost) / (unsigned)(d.late + rest));
        d.late += rest;
      }
    }
    return t;
  }
  Deal t{d.pos < level ? lo + d.pos : lo + ahead, lo + ahead, level, 0, lo + n, d.W};
  d.gap -= rounds * cost;
  if (rounds && d.gap <= 0) {        // the late ones now have less, or as much
    d.pos -= level;
    if (d.pos < 0) d.pos += d.W;
    d.late = level;
    d.gap = -d.gap;
  }
  t.at2 = lo + ahead + d.pos;
  if (more) {
    const int rest = (int)((unsigned)(n - ahead) % (unsigned)d.W);
    if (rest) {
      d.pos -= rest;
      if (d.pos < 0) d.pos += d.W;
      d.late = rest;
      d.gap = cost;
    }
  }
  return t;
}

}  // namespace mlc
