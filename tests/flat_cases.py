"""Step sizes that take the flattened layout (the CPU test asks the library's
host code, the GPU test compares results)."""
FLAT = [dict(K=6000, M=37, T=97, noise_kind=1), dict(K=22000, M=22, T=98, noise_kind=1, B=2.0),  # 13 samples a workgroup
        dict(K=6000, M=37, T=97, noise_kind=2, jump_prob=0.1, jump_size=0.4, alpha=0.5), dict(K=3001, M=100, T=64),
        dict(K=1100, M=257, T=30), dict(K=1100, M=300, T=30, alpha=0.5)]
# 9000 * 19 * 97 state steps, 9 of 256 lanes idle: 1.8 us of a full device (and one launch with a handle)
PER_SAMPLE = [dict(K=9000, M=19, T=97, noise_kind=1), dict(K=17000, M=64, T=60)]
# Impulses on the caller's memory: samples of five waves that all start at once, long horizons among many obstacles
IMPULSE = {(86, 274, 300, 200): False, (86, 124, 300, 200): True, (86, 125, 300, 200): False, (508, 270, 257, 65): True,
           (507, 270, 257, 65): True, (503, 270, 257, 65): False, (86, 249, 319, 65): True, (86, 250, 319, 65): False,
           (86, 274, 320, 200): True, (86, 600, 300, 64): True, (30, 270, 256, 200): False}  # (K, T, M, n_obs): flattened
