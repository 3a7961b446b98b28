/* Generated by gen_exp2_fit.py -- do not edit.
 * 2^f = 1 + f E(f), |f| <= 1/2: Chebyshev interpolant of E, ascending powers of f.
 * Maximum relative error in double precision: 1.56e-16.
 */
#pragma once

namespace rbe2d {

constexpr int kExp2Terms = 11;
constexpr double kExp2[kExp2Terms] = {
    0.6931471805599453,
    0.24022650695910097,
    0.0555041086648216,
    0.009618129107606888,
    0.0013333558146416936,
    0.0001540353044173605,
    1.525273382983612e-05,
    1.321544258792169e-06,
    1.0178062445845774e-07,
    7.072585949269223e-09,
    4.4549605981865186e-10,
};

}  // namespace rbe2d
