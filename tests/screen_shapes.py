"""Searches at the edges of the screening pass, for the tests of its route (on
the CPU) and of its results (on a GPU): which the library screens, and why not."""

VGOS = [b + 32.0 * i for b in (3000.0, 5240.0, 6360.0, 10200.0) for i in range(8)]
LATTICES = {
    "1if": [3000.0],
    "3if-spread": [3000.0, 3032.0, 5240.0],
    "16if-compact": [3000.0 + 32.0 * i for i in range(16)],
    "8if-compact": [3000.0 + 32.0 * i for i in range(8)],
    "5if-compact": [3000.0 + 32.0 * i for i in (0, 1, 2, 3, 6)],
    "17if": VGOS[:17],
    "20if-even": [3000.0 + 64.0 * i for i in range(19)] + [3032.0],   # 19 even positions, 1 odd
    "32if-vgos": VGOS,
}
WINDOWS = [1, 2, 5]
K, N_DM = 70, 80   # 13760 segments

# (lattice, channels, sbd_pad, rates, precision): screened
SCREENED = [
    ("1if", 32, 4, 2, "f32"), ("3if-spread", 64, 1, 4, "f32"), ("16if-compact", 32, 8, 2, "f32"),
    ("5if-compact", 16, 8, 1, "f32"), ("17if", 32, 2, 4, "f32"), ("20if-even", 64, 2, 3, "f32"),
    ("32if-vgos", 64, 4, 8, "f32"), ("32if-vgos", 16, 4, 9, "f32"), ("20if-even", 128, 2, 4, "f32"),
    ("32if-vgos", 128, 4, 3, "f32"), ("16if-compact", 256, 4, 4, "f32"), ("3if-spread", 256, 1, 1, "f32"),
    ("3if-spread", 16, 8, 64, "f32"),
    ("16if-compact", 32, 8, 2, "f16x3"), ("3if-spread", 64, 1, 8, "f16x3"), ("17if", 32, 2, 4, "f16x3"),
    ("20if-even", 64, 2, 4, "f16x3"), ("32if-vgos", 64, 4, 1, "f16x3"), ("32if-vgos", 128, 4, 1, "f16x3"),
    ("16if-compact", 256, 4, 1, "f16x3"),
    ("17if", 32, 8, 4, "f16"), ("32if-vgos", 64, 4, 4, "f16"), ("32if-vgos", 64, 4, 8, "f16"),
    ("32if-vgos", 16, 8, 16, "f16"),
]
# evaluated whole: too few units for the form, or a shape the pass does not have
WHOLE = [
    ("5if-compact", 16, 4, 1, "f32"), ("3if-spread", 32, 4, 1, "f32"), ("3if-spread", 256, 4, 2, "f32"),
    ("8if-compact", 32, 4, 1, "f16x3"), ("16if-compact", 16, 8, 1, "f16x3"), ("3if-spread", 32, 4, 2, "f16x3"),
    ("8if-compact", 128, 1, 2, "f16x3"),
    ("32if-vgos", 64, 4, 1, "f16"), ("32if-vgos", 64, 8, 1, "f16"), ("17if", 32, 4, 2, "f16"),
    ("16if-compact", 64, 4, 8, "f16"), ("20if-even", 64, 4, 8, "f16"), ("32if-vgos", 128, 4, 8, "f16"),
]
PRECISION = {"f32": 0, "f16x3": 1, "f16": 2}
