// Matrices whose weak planes the eight-product form (qgemm8_kern.hpp) would lose.
//
// The form adds planes before it multiplies, so its rounding errors are relative to the norm of all four planes; the direct form's
// are relative to the terms of each output plane.  The two differ where planes stay separate in a solve, that is in and near the
// three complex subalgebras span(1, i), span(1, j), span(1, k) and their cosets: the planes in two pairs, {s, x | y, z},
// {s, y | x, z} or {s, z | x, y}.  There an output plane of one pair takes products within the pairs and one of the other pair
// products across them, so that a weak pair's outputs have a weak factor in every term.  A matrix keeps the direct form if one
// pair of a pairing is weak against the other: below 1/5 of it over the whole matrix (Frobenius norms), or below 1/16 in one row.
// (Blocks that no product couples show in their rows; over rows that are coupled the weak pair fills up, so that one row alone
// need not reach the whole matrix's ratio.)
//
// Where the lines lie, from products of iid planes with the two pairs at a ratio r (K = 256, FP32, sequential sums), errors of the
// weak planes by the eight-product form over those by the direct form: r = 1: 0.7, 0.5: 0.9, 0.35: 1.2, 0.2: 1.8, 0.1: 3.6,
// 1/16: 6, and in proportion to 1/r below; the error in the norm of all planes is 0.6 to 0.9 of the direct form's throughout.
// What stays exact in both forms keeps the eight products: matrices with one plane, and those with planes (s, x) or (y, z) alone
// whose two planes are of like size.  That holds for the multiples of A^H that a solve starts from; with a start of the caller's,
// whose other planes the direct form lets vanish, such matrices keep the direct form too.
#pragma once

namespace qp {

// squared ratios of the whole matrix and of a row
constexpr double kPairRatio = 1.0 / 25, kRowPairRatio = 1.0 / 256;

// What a matrix or a row is, as flags to be united: planes 0..3 that are not zero in bits 0..3,
constexpr unsigned kPlanesWeak = 16, kPlanesApart = 32;  // one pair weak against the other; planes apart, and exact in both forms

// s, x, y, z: the planes' sums of squares; bit p of `nonzero`: plane p has an element that is not zero (its square may be)
__host__ __device__ inline unsigned plane_flags(double s, double x, double y, double z, unsigned nonzero, double ratio) {
  auto weak = [&](double u, double v) { return (u < v ? u : v) <= ratio * (u < v ? v : u); };
  if (nonzero == 0) return 0;
  if ((nonzero & (nonzero - 1)) == 0) return kPlanesApart;
  if ((nonzero & 3) == 0 || (nonzero & 12) == 0) return weak(s + y, x + z) ? kPlanesWeak : kPlanesApart;
  return weak(s + x, y + z) || weak(s + y, x + z) || weak(s + z, x + y) ? kPlanesWeak : 0;
}

}  // namespace qp
