"""The library's launch rules, restated for the tests that ask for a certain launch."""


def select_shape(H, n_qb, n_kb):
    """Slots per lane and (waves, rows per wave) of the selection's workgroups: the fewest rounds of workgroups over
    256 compute units times the time of one (hundredths of 8 one-row waves); up to 2 slots also two workgroups of 8
    two-row waves at once."""
    for lim, cpl in ((128, 2), (256, 4), (384, 6), (512, 8), (768, 12), (1088, 17), (1536, 24), (2304, 36), (4096, 64)):
        if n_kb <= lim:
            break
    if cpl > 17:
        return cpl, ((4, 1) if cpl == 64 else (8, 1))

    def rounds(rows):
        return -(-(H * -(-n_qb // rows)) // 256)

    options = [((8, 1), 100 * rounds(8)), ((4, 1), 90 * rounds(4)), ((12, 1), 112 * rounds(12)), ((16, 1), 127 * rounds(16))]
    if cpl <= 6:
        options.append(((12, 2), 210 * rounds(24)))
    if cpl <= 2:
        options.append(((8, 2), rounds(16) // 2 * 215 + rounds(16) % 2 * 135))
    return cpl, min(options, key=lambda o: o[1])[0]  # the first of equals


def attn_groups(H, n_qb, n_kb, bq, bk):
    """Key groups per query block of the attention, by rows and by 64-key chunks per head."""
    rows, chunks = H * n_qb, n_kb * (bk // 64)
    if rows <= 256 and chunks >= 64:
        return 4
    least = 7 if rows <= 512 else 64 if bq == 128 else 32
    return 2 if rows <= 3072 and chunks >= least else 1
