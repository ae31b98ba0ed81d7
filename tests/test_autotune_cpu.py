"""Autotune cache bookkeeping (no GPU: a stand-in solver reports timings)."""
from paper_1708_07525_amd import autotune


class FakeSolver:
    def __init__(self, nx, ny, precision="fp32"):
        self.nx, self.ny, self.precision = nx, ny, precision
        self.tile = (256, 1)
        self.policy = -1
        self.timed = 0

    def autotune(self, steps):
        self.timed += 1
        self.tile = (128, 2)
        self.policy = 1
        return self.tile, 0.25

    def set_tile(self, tx, ty):
        self.tile = (tx, ty)

    def set_cache_policy(self, p):
        self.policy = p

    def get_cache_policy(self):
        return self.policy

    def set_steps_per_launch(self, n):
        self.spl = n

    def get_steps_per_launch(self):
        return getattr(self, "spl", 2)

    def set_strip_width(self, n):
        self.strip = n

    def get_strip_width(self):
        return getattr(self, "strip", 4)

    def set_tile_rows(self, n):
        self.rows = n

    def get_tile_rows(self):
        return getattr(self, "rows", 12)


def test_size_class_and_key():
    assert [autotune.size_class(n) for n in (1, 3, 64, 65, 2048)] == [1, 4, 64, 128, 2048]
    g = f"g{autotune.KERNEL_GENERATION}"
    assert autotune.key("MI355X", "fp32", 100, 200, True) == g + "|MI355X|fp32|128x256|field"
    assert autotune.key("MI355X", "fp32", 100, 200, True, node_walls=True) == g + "|MI355X|fp32|128x256|field|node-walls"


def test_tune_times_once_per_class(tmp_path):
    path = str(tmp_path / "cache.json")
    a = FakeSolver(100, 100)
    assert autotune.tune(a, "gpu", False, path=path) == ((128, 2), 0.25)
    assert a.timed == 1
    b = FakeSolver(120, 90)          # same class: 128x128, uniform, fp32
    b.tile = (64, 8)
    assert autotune.tune(b, "gpu", False, path=path) == ((128, 2), None)
    assert b.timed == 0 and b.tile == (128, 2) and b.policy == 1 and b.strip == 4 and b.rows == 12
    c = FakeSolver(120, 90, "fp16s")  # other precision: timed again
    autotune.tune(c, "gpu", False, path=path)
    assert c.timed == 1
    assert len(autotune.load(path)) == 2


def test_corrupt_cache_is_ignored(tmp_path):
    path = tmp_path / "cache.json"
    path.write_text("{not json")
    s = FakeSolver(64, 64)
    autotune.tune(s, "gpu", True, path=str(path))
    assert s.timed == 1 and autotune.load(str(path))


def test_wall_families_are_tuned_apart(tmp_path):
    path = str(tmp_path / "cache.json")
    a = FakeSolver(100, 100)
    autotune.tune(a, "gpu", False, path=path)
    b = FakeSolver(100, 100)
    autotune.tune(b, "gpu", False, path=path, node_walls=True)
    assert a.timed == 1 and b.timed == 1 and len(autotune.load(path)) == 2


class LaunchSolver(FakeSolver):
    """A stand-in whose lattices of 1500 columns and more march by default, while nothing else is set;
    tuned to the default launch (fastest == "march") or to a tile."""

    def __init__(self, nx, ny, fastest):
        super().__init__(nx, ny)
        self.fastest = fastest
        self.defaults()

    def defaults(self):
        self.tile, self.policy, self.spl, self.strip, self.rows = (0, 0), -1, 0, -1, 0

    def get_region_steps(self):
        return 0

    def get_march_steps(self):
        at_default = (self.tile, self.policy, self.spl, self.strip, self.rows) == ((0, 0), -1, 0, -1, 0)
        return 4 if self.nx >= 1500 and at_default else 0

    def autotune(self, steps):
        self.timed += 1
        self.defaults()
        if self.fastest != "march":
            self.tile, self.policy, self.spl, self.strip, self.rows = (128, 2), 1, 3, 8, 12
        return self.tile, 0.25


def test_a_set_solver_is_tuned_under_its_lattices_key(tmp_path):
    """What the caller has set before does not choose the cache entry: a 1100^2 lattice, which does not
    march, keeps its own entry beside that of a 2048^2 lattice of its size class, which does."""
    path = str(tmp_path / "cache.json")
    a = LaunchSolver(2048, 2048, "march")
    a.set_steps_per_launch(2)                   # set by the caller before
    assert autotune.tune(a, "gpu", False, path=path)[1] == 0.25 and a.get_march_steps() == 4
    small = LaunchSolver(1100, 1100, "tile")
    assert autotune.tune(small, "gpu", False, path=path)[1] == 0.25 and small.timed == 1
    assert small.spl == 3 and len(autotune.load(path)) == 2
    b = LaunchSolver(2048, 2048, "march")
    b.set_steps_per_launch(1)                   # a slow setting does not stay
    assert autotune.tune(b, "gpu", False, path=path)[1] is None and b.timed == 0 and b.get_march_steps() == 4
    other = LaunchSolver(1100, 1100, "tile")
    assert autotune.tune(other, "gpu", False, path=path)[1] is None and other.spl == 3 and other.rows == 12
    assert autotune.tune(b, "gpu", False, path=path, force=True)[1] == 0.25 and b.timed == 1
    assert len(autotune.load(path)) == 2


def test_an_entry_of_another_launch_is_timed_again(tmp_path):
    """An entry that names a launch which this lattice does not take by default is not applied."""
    path = str(tmp_path / "cache.json")
    k = autotune.key("gpu", "fp32", 1100, 1100, False)
    autotune.store({k: {"tile": [256, 1], "launch": "march"}}, path)
    s = LaunchSolver(1100, 1100, "tile")
    assert autotune.tune(s, "gpu", False, path=path)[1] == 0.25 and s.timed == 1 and s.spl == 3
    assert autotune.load(path)[k]["launch"] == ""
