"""Which weight-gradient tile a batch-block-32 layer takes, and in how many
splits, written out from the rules stated in the library's sources: tests use
it to hold the layers they are meant for."""

BITS = {0: 8, 1: 4, 2: 6, 3: 6}


def _out(cv):
    return ((cv["h"] + 2 * cv["ph"] - cv["kh"]) // cv["sh"] + 1, (cv["w"] + 2 * cv["pw"] - cv["kw"]) // cv["sw"] + 1)


def one_tap_splits(cv, fg, fx):
    ho, wo = _out(cv)
    gb, xb = -(-cv["cout"] // 32), -(-cv["cin"] // 32)
    tiles = cv["kh"] * cv["kw"] * ((gb + 1) // 2) * ((xb + 1) // 2)
    pairs = (cv["n"] // 32 * ho * wo + 1) // 2
    single = gb == xb == 1 and fg == fx and fg in (0, 1)
    return max(1, min(1280 // tiles, pairs // 32) if single else min(512 // tiles, pairs // 16))


def row_plan(cv, fg, fx):
    """(tile side in 32-row blocks, splits in all) of the kernel-row tile, or
    None: another kernel serves the layer."""
    if cv["n"] % 32 or cv["kw"] != 3 or cv["sw"] not in (1, 2):
        return None
    ho, wo = _out(cv)
    ng, gb, xb = cv["n"] // 32, -(-cv["cout"] // 32), -(-cv["cin"] // 32)
    fit = 0x7FFFFF00 // max(ho * wo * gb * 128 * BITS[fg], cv["h"] * cv["w"] * xb * 128 * BITS[fx])
    # the padded width of a row fits the offsets, too
    if fit == 0 or (wo + 3) * max(gb * 128 * BITS[fg], cv["sw"] * xb * 128 * BITS[fx]) >= 0x7FFFF000:
        return None
    launches = -(-ng // fit)                 # each below 2 GiB of codes
    if launches > 1 and (gb > 1 or xb > 1):
        return None
    total = (-(-ng // launches) * ho + 1) // 2 * wo
    part = 32 * gb * cv["kh"] * 3 * 32 * xb * 4

    def tiles(k):
        return cv["kh"] * -(-gb // k) * -(-xb // k)

    def split(k):
        return max(1, min((256 if k == 2 else 512) // tiles(k), total // 24, (16 << 20) // part // launches))

    nb = 1
    if gb > 1 or xb > 1:
        cols = total // (4 * split(2)) if gb > 1 and xb > 1 else 0
        fills = split(2) * tiles(2) >= 224 or cols >= 64
        if fg == 0:
            nb = 2 if cols >= 12 and fills else 1
        elif cv["sw"] == 1 and cols >= (16 if BITS[fx] == 6 else 24):
            nb = 2 if fills else 1
        elif total > 128:
            return None
    return (nb, split(nb) * launches) if split(nb) * launches <= max(1, (16 << 20) // part) else None


def workspace_bytes(cv, fg, fx):
    plan = row_plan(cv, fg, fx)
    splits = plan[1] if plan else one_tap_splits(cv, fg, fx)
    part = 4 * 32 * -(-cv["cout"] // 32) * cv["kh"] * cv["kw"] * 32 * -(-cv["cin"] // 32)
    return splits * part if splits > 1 else 0
