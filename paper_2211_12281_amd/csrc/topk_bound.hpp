// Roundings that the ranking's check counts against the sums of the scan (plain C++).
//
// bf16 rows: the products are exact, d sums; each is off by at most 2^-23 of what it holds, |a| |b| at most (2^-24 if it is rounded to
// nearest, 2^-23 if it is truncated: the count does not rely on which).  fp32 rows: two fp16 pieces of every element and three of the four
// products of pieces, so three sums per element, and the pieces themselves: an element is off by at most 2^-23 of it (24 bits as 11 + 11 and a sign), either
// factor by one unit, and the product of the lower pieces, left out, is 2^-22 of the product at most: four units, and eight are counted
// (elements below 2^-16 of their row's largest are off by 2^-40 of that instead: d 2^-40 |a| |b| in all).
#pragma once

constexpr int TK_PIECES = 8;

// sum of d products a_j b_j: units of 2^-23 |a| |b|
constexpr int topk_product_units(int d, bool bf16) { return bf16 ? d : 3 * d + TK_PIECES; }

// 2 q.t - |t|^2: units of 2^-22 (|q| + |t|)^2.  2 |q| |t| is at most half the square, so the three sums per element of fp32 rows are 3/4 of
// a unit; the rest is for the norms' own sums (chains of d / 8, rounded to nearest) and the start value.
constexpr int topk_distance_units(int d, bool bf16) { return d + 2 + (bf16 ? 0 : TK_PIECES); }
