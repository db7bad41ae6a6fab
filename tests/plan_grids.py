"""Grids of the launch-path tests that a rule of the library has to send to a certain
kernel on 256 compute units: test_host_runtime.py checks that it does,
test_gpu_paths.py what the kernel computes."""

# full-round D2Q9 marches with cached stores, at every pass limit but those listed
CACHED_2D = [(14989, 3), (13043, 123), (6350, 269), (16323, 7)]
CACHED_2D_HALF = [((13043, 123), 4)]

# D3Q19 passes on grids with an axis shorter than a tile's halo: by the tall tiles of the
# march, and by the 8-row tiles that are faster on few planes and on rows of columns
FLAT_3D = [(1200, 900, 1), (1000, 800, 2), (301, 299, 3), (3, 300, 300), (1, 700, 200),
           (60, 2, 9000), (3, 5, 10000), (2, 900, 500), (500, 4, 500)]
FLAT_3D_8_ROWS = [(303, 154, 3), (399, 138, 4), (300, 3, 300), (1020, 4, 200), (180, 4, 1200)]

# D3Q19 grids where two single steps take less than a pass
SINGLE_3D = [(1, 1, 65535), (2, 1, 30000), (4, 4, 20000), (50000, 4, 4), (600, 600, 1)]
