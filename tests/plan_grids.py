"""Grids of the launch-path tests that a rule of the library has to send to a certain
kernel on 256 compute units: test_host_runtime.py checks that it does,
test_gpu_paths.py what the kernel computes."""

# full-round D2Q9 marches with cached stores, at every pass limit but those listed
CACHED_2D = [(14989, 3), (13043, 123), (6350, 269), (16323, 7)]
CACHED_2D_HALF = [((13043, 123), 4)]

# D3Q19 passes on grids with an axis shorter than a tile's halo
FLAT_3D = [(600, 600, 1), (512, 512, 2), (301, 299, 3), (3, 300, 300), (1, 700, 200),
           (300, 3, 300), (60, 2, 9000), (4, 4, 20000), (2, 1, 30000), (1, 1, 9000)]
