// Generated by fit_minimax.py -- coefficients in increasing powers of s.
#pragma once
// ATAN_SMALL_POLY: max relative error 3.023e-08 (mean +3.8e-09) on s = u^2 in [0, 1/3], float32 coefficients
#define ATAN_SMALL_POLY_DEGREE 5
static constexpr double ATAN_SMALL_POLY_D[6] = {1.0, -0.3333298711841056, 0.19984731859998758, -0.14063327855665328, 0.0964722545709791, -0.043257934159236};
// ATAN_UNIT_POLY: max relative error 1.919e-08 (mean +5.7e-10) on s = u^2 in [0, 1], float32 coefficients
#define ATAN_UNIT_POLY_DEGREE 8
static constexpr double ATAN_UNIT_POLY_D[9] = {1.0, -0.33333152636378494, 0.199937699897483, -0.14211028149100122, 0.10665882858518054, -0.07551924459925496, 0.04320809492563086, -0.016365406217941064, 0.0029200115816710123};
// ATANH_POLY: max relative error 2.298e-08 (mean +5.2e-10) on s = v^2 in [0, 1/4], float32 coefficients
#define ATANH_POLY_DEGREE 5
static constexpr double ATANH_POLY_D[6] = {1.0, 0.3333373095973716, 0.19978174446377814, 0.1466972156549513, 0.08240611709836752, 0.18179634965763014};
