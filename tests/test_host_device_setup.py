"""What the library's device set-up does when a device allocation or an upload
fails: the call returns an error, gives back what it had allocated, and works
when it is called again.  Kernels take the set-up's pointers unchecked, so a
failure that went unseen would be a GPU fault.  Runs on the CPU: the HIP
runtime calls of libmfgmg.so are those of tests/native/hip_host.cpp (host
memory, kernels never run), in a process of its own."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# base level, boundary condition, element and refined cells: uniform levels,
# levels run as a grid through maps, blocks and hanging nodes, lattice levels
CASES = {"uniform": (3, "dirichlet", 1, ()), "noflux": (3, "noflux", 1, ()),
         "adaptive": (3, "dirichlet", 1, ((0, 0, 0), (5, 2, 7))), "q3": (3, "dirichlet", 2, ())}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    so = str(tmp_path_factory.mktemp("hip_host") / "hip_host.so")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC",
                        os.path.join(ROOT, "tests", "native", "hip_host.cpp"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return so


def run(stub, what, case):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, what, case], capture_output=True, text=True,
                       timeout=300, cwd=ROOT)
    assert r.returncode == 0, f"{what} {case}: exit {r.returncode}\n{r.stdout}\n{r.stderr}"


@pytest.mark.parametrize("case", sorted(CASES))
def test_failed_allocation_is_reported(stub, case):
    run(stub, "allocation", case)


@pytest.mark.parametrize("case", sorted(CASES))
def test_failed_upload_is_reported(stub, case):
    run(stub, "upload", case)


def test_failed_allocation_of_local_levels_is_reported(stub):
    run(stub, "local", "adaptive")

@pytest.mark.parametrize("case", sorted(CASES))
def test_host_memory_running_out_is_reported(stub, case):
    """No C++ exception leaves the C entries that set up device data."""
    run(stub, "host_memory", case)

@pytest.mark.parametrize("case", sorted(CASES))
def test_viscosity_that_failed_half_way_is_not_used(stub, case):
    """A later mfgmg_set_viscosity that fails after it began to change the levels leaves no mix of two viscosities
    behind (the 4^3 level's matrix and the coarse factor of the old one under the operators of the new one): calls
    that need it say that none is set.  One that fails before leaves the old one in use."""
    run(stub, "half_way", case)

def test_uniform_leaf_uploads_no_cell_tables(stub):
    """No kernel reads cell or block tables of a uniform leaf; building and uploading them was three quarters of its
    set-up.  What it does upload is the constrained dofs (8 bytes each), the pressure lattice (4 bytes a point), the
    cells whose mean a coarser cell takes (8 x 4 bytes) and the tables of the two smallest levels."""
    run(stub, "uniform_tables", "uniform")


# ---------------------------------------------------- the process with the stub

class Child:
    def __init__(self, stub, case):
        import numpy as np
        self.np = np
        self.hip = C.CDLL(stub, mode=C.RTLD_GLOBAL)   # before the library: found first
        for f in ("stub_mallocs", "stub_copies", "stub_news", "stub_uploaded", "stub_held"):
            getattr(self.hip, f).restype = C.c_int64
        for f in ("stub_fail_malloc", "stub_fail_copy", "stub_fail_new"):
            getattr(self.hip, f).argtypes = [C.c_int64]
        sys.path.insert(0, ROOT)
        from paper_1907_06696_amd import mfgmg
        self.m = mfgmg
        self.spec = CASES[case]

    def solver(self):
        base, bc, k, refined = self.spec
        s = self.m.Solver(base)
        s.set_boundary(bc)
        s.set_element(k)
        if refined:
            s.refine(self.np.array([(base,) + c for c in refined], self.np.int32), 1)
        s.finalize_mesh()
        self.mu = self.np.ones(s.leaf_quadrature_points().shape[:2])
        return s

    def set_viscosity(self, s):
        return s.lib.mfgmg_set_viscosity(s.h, self.mu.ctypes.data, None)

    def every_failure(self, arm, counter, prepare, call):
        """Counts the operations of a call that succeeds, then has each of them fail in turn."""
        hip, m = self.hip, self.m
        s = prepare()
        arm(0)
        assert call(s) == m.OK
        count, kept = counter(), hip.stub_held()
        s.close()
        assert count > 0 and hip.stub_held() == 0
        for n in range(1, count + 1):
            s = prepare()
            arm(n)
            code = call(s)
            arm(0)
            assert code in (m.ERR_NOMEM, m.ERR_HIP), f"operation {n} of {count} failed and the call returned {code}"
            # called again, it finds nothing half done and nothing kept twice
            assert call(s) == m.OK and hip.stub_held() == kept, f"after failure {n} of {count}"
            s.close()
            assert hip.stub_held() == 0

    def allocation(self):
        self.every_failure(self.hip.stub_fail_malloc, self.hip.stub_mallocs, self.solver, self.set_viscosity)

    def upload(self):
        self.every_failure(self.hip.stub_fail_copy, self.hip.stub_copies, self.solver, self.set_viscosity)

    def host_memory(self):
        np, hip, m = self.np, self.hip, self.m
        f = np.zeros(self.solver().leaf_quadrature_points().shape)

        def rhs(s):
            b = np.zeros(s.info()["n_u"][s.info()["L"]])
            return s.lib.mfgmg_assemble_rhs(s.h, f.ctypes.data, b.ctypes.data, None)

        calls = [(self.solver, self.set_viscosity), (self.solver, rhs)]
        if self.spec[3]:
            calls.append((self.ready, self.vcycle_local))
        for prepare, call in calls:
            s = prepare()
            hip.stub_fail_new(0)
            assert call(s) == m.OK
            count = hip.stub_news()
            s.close()
            for n in sorted({1, 2, 3, count, *(max(1, int(count * q / 40)) for q in range(40))}):
                s = prepare()
                hip.stub_fail_new(n)
                code = call(s)
                hip.stub_fail_new(0)
                assert code == m.ERR_NOMEM, f"host allocation {n} of {count} failed and the call returned {code}"
                assert call(s) == m.OK
                s.close()
                assert hip.stub_held() == 0

    def half_way(self):
        np, hip, m = self.np, self.hip, self.m
        s = self.ready()
        L = s.info()["L"]
        x, y = (np.zeros(s.info()["n_u"][L]) for _ in range(2))

        def vmult():
            return s.lib.mfgmg_vmult(s.h, L, m.FP64, x.ctypes.data, y.ctypes.data, None)

        hip.stub_fail_new(0)
        assert self.set_viscosity(s) == m.OK
        count = hip.stub_news()
        for n in sorted({1, count // 2, count}):   # host tables of the eigenvalue estimates to the pressure's
            hip.stub_fail_new(n)
            assert self.set_viscosity(s) == m.ERR_NOMEM
            hip.stub_fail_new(0)
            assert vmult() == m.ERR_STATE, f"host allocation {n} of {count}"
            assert self.set_viscosity(s) == m.OK and vmult() == m.OK
        for n in (1, 2):   # its temporary arrays, before it changes anything
            hip.stub_fail_malloc(n)
            assert self.set_viscosity(s) != m.OK
            hip.stub_fail_malloc(0)
            assert vmult() == m.OK
        self.mu[0, 0] = -1.0
        assert self.set_viscosity(s) == m.ERR_INVALID and vmult() == m.OK
        s.close()

    def uniform_tables(self):
        self.spec = (5, "dirichlet", 1, ())
        s = self.solver()
        before = self.hip.stub_uploaded()
        assert self.set_viscosity(s) == self.m.OK
        i = s.info()
        constrained = sum(i["n_u"]) - sum(i["n_free"])
        bound = 8 * constrained + 4 * i["n_p"] + 4 * sum(i["n_cells"][2:]) + 128 * 1024
        assert self.hip.stub_uploaded() - before <= bound
        s.close()

    def ready(self):
        s = self.solver()
        assert self.set_viscosity(s) == self.m.OK
        return s

    def vcycle_local(self, s):
        b, x = (self.np.zeros(s.info()["n_u"][s.info()["L"]]) for _ in range(2))
        return s.lib.mfgmg_vcycle_local(s.h, self.m.FP64, b.ctypes.data, x.ctypes.data, None)

    def local(self):
        self.every_failure(self.hip.stub_fail_malloc, self.hip.stub_mallocs, self.ready, self.vcycle_local)
        self.every_failure(self.hip.stub_fail_copy, self.hip.stub_copies, self.ready, self.vcycle_local)


if __name__ == "__main__":
    child = Child(sys.argv[1], sys.argv[3])
    getattr(child, sys.argv[2])()
