"""The stepped MFMA kernel's launch-shape rule, and the choice among the kernels above 128 batch rows,
stated independently of the library's host code so that tests can check the library against it."""

# Per-step time of a workgroup (us per step of 256 k) with t batch tiles: fixed + tile * t, for
# 64- and 128-row workgroups, and the extra cost of two K parts (us), per kind of
# dequantization: register tables (fitted 4-bit codebooks), the 4-bit LDS table (any other
# 4-bit codebook) and 8-bit codes.
COSTS = {
    "register": (0.376, 0.184, 0.500, 0.300, 5.0),
    "table4": (0.283, 0.198, 0.205, 0.374, 3.1),
    "bits8": (0.422, 0.279, 0.156, 0.600, 3.0),
}


def stepped_shape(m, k, n, kind="register"):
    return _stepped(m, k, n, kind)[0]


def _stepped(m, k, n, kind):
    """((64-row workgroups, batch tiles per workgroup column, K parts), its cost in us or None where none fits). Every shape whose grid
    has at most 256 workgroups competes on (steps per workgroup) x (per-step time), plus the
    cost of two K parts (allowed from 16 steps of 256); t runs t0, ceil(t0 / 2), ... 1 with
    t0 = min(ceil(m / 16), cap), cap 8 for register tables and 4 otherwise; 8-bit codes never
    take 128-row workgroups with one tile. With no shape that fits: 128-row workgroups with t0
    tiles, unless 64-row ones fit."""
    f64, t64, f128, t128, two = COSTS[kind]
    cap = 8 if kind == "register" else 4
    t0 = min(-(-m // 16), cap)
    gy = -(-m // (16 * cap)) if m > 16 * cap else 1
    best, best_cost = ((-(-n // 64)) * gy <= 256, t0, 1), None
    steps = -(-k // 256)
    for rows in (128, 64):
        t = t0
        while True:
            for parts in ((1, 2) if steps >= 16 else (1,)):
                if kind == "bits8" and rows == 128 and t == 1:
                    continue     # left out for 8-bit codes
                if -(-n // rows) * -(-m // (16 * t)) * parts > 256:
                    continue
                per = f128 + t128 * t if rows == 128 else f64 + t64 * t
                cost = -(-steps // parts) * per + (two if parts == 2 else 0.0)
                if best_cost is None or cost < best_cost:
                    best, best_cost = (rows == 64, t, parts), cost
            if t == 1:
                break
            t = (t + 1) // 2
    return best, best_cost


def stepped_name(m, k, n, kind="register"):
    narrow, t, _ = stepped_shape(m, k, n, kind)
    bits = 8 if kind == "bits8" else 4
    pairs = "false" if kind == "register" else "true"
    coal = "true" if t <= 2 else "false"
    if narrow:
        return f"k_mfma2_narrow<{bits}, {t}, {pairs}, {coal}>"
    return f"k_mfma2<{bits}, {t}, 4, {pairs}, {coal}>"


# Prefill kernel, us: a launch, a round of 256 workgroups, a step of 64 k with 1 .. 4 batch tiles of
# 64 rows (per round, and per tile and full chip), an output; two K parts, an output of those, more
# of it where rows of y are not whole cache lines.
PREFILL_US = {
    4: (2.5, 2.1, (0.561, 0.655, 0.879, 1.095), 0.119, 0.65e-6, 0.98, 5.35e-6, 1.9e-6),
    8: (3.3, 2.0, (0.995, 1.138, 1.501, 1.712), 0.081, 0.59e-6, 0.96, 5.35e-6, 2.0e-6),
}
# Stepped kernel beside the others: a launch, the factor on its model, more of it for every further
# XCD (of 7) that fetches the codes of a row block and for rows that are not whole cache lines of
# 128 bytes, two K parts, an output. K-quartered kernels: a round of 256 workgroups, a step of
# 128 k per round, more of it likewise, a step of a full chip.
STEPPED_US = {
    "register": (4.1, 0.956, 0.169, 0.017, 11.4, 1.16e-6),
    "table4": (5.4, 0.935, 0.234, 0.054, 2.9, 1.1e-6),
    "bits8": (5.6, 0.875, 0.588, 0.136, 5.25, 1.125e-6),
}
QUARTERED_US = {4: (10.8, 0.797, 0.366, 0.03, 0.2), 8: (8.84, 1.475, 0.152, 0.0, 0.434)}


def code_fetches(gx, gy):
    """XCDs among 0 .. 7 on which workgroups 0, gx, 2 gx .. (gy - 1) gx land, round-robin."""
    return len({y * gx % 8 for y in range(min(gy, 8))})


def prefill_shape(m, k, n, bits):
    """(batch tiles, K parts) of the prefill kernel and its cost."""
    launch, rnd, step, full, out, two, two_out, two_partial = PREFILL_US[bits]
    two_out += two_partial if n % 32 else 0.0
    steps, best = -(-k // 64), None
    for parts in (1, 2) if steps >= 2 else (1,):
        for bt in (1, 2, 3, 4):
            wgs = -(-m // (64 * bt)) * -(-n // 256) * parts
            rounds = -(-wgs // 256)
            cost = (launch + rnd * rounds
                    + -(-steps // parts) * (step[bt - 1] * rounds + full * bt * wgs / 256)
                    + out * m * n + (two + two_out * m * n if parts == 2 else 0.0))
            if best is None or cost < best[1]:
                best = (bt, parts), cost
    return best


def wide_costs(m, k, n, kind="register"):
    """Cost in us of every kernel that serves a call of more than 128 rows, by path name."""
    bits = 8 if kind == "bits8" else 4
    partial = k * bits // 8 % 128 != 0
    costs = {}
    (narrow, tiles, parts), model = _stepped(m, k, n, kind)
    if model is not None:
        launch, step, spread, part, two, out = STEPPED_US[kind]
        fetches = code_fetches(-(-n // (64 if narrow else 128)), -(-m // (16 * tiles)))
        model -= COSTS[kind][4] if parts == 2 else 0.0
        costs["mfma"] = (launch + model * (step + spread * (fetches - 1) / 7 + part * partial)
                         + (two if parts == 2 else 0.0) + out * m * n)
    if (kind == "register" and n >= 4096) or (bits == 8 and n >= 16384):
        rnd, step, spread, part, full = QUARTERED_US[bits]
        gx, gy, steps = -(-n // 128), -(-m // 128), -(-k // 128)
        each = step + spread * (code_fetches(gx, gy) - 1) / 7 + part * partial
        costs["mfma_kq"] = -(-gx * gy // 256) * (rnd + steps * each) + steps * full * gx * gy / 256
    if k < 1 << 22 and n < 1 << 21 and -(-m // 64) * -(-n // 256) < 1 << 23:
        costs["mfma_pf"] = prefill_shape(m, k, n, bits)[1]
    return costs


def wide_name(m, k, n, kind="register"):
    bits = 8 if kind == "bits8" else 4
    costs = wide_costs(m, k, n, kind)
    path = min(costs, key=costs.get) if costs else "mfma"
    if path == "mfma":
        return stepped_name(m, k, n, kind)
    if path == "mfma_kq":
        return "k_mfma_kq" if bits == 4 else "k_mfma_kq8"
    return f"k_mfma_pf<{bits}, {prefill_shape(m, k, n, bits)[0][0]}>"
