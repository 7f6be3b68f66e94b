"""Host rules of the launch shapes, worked through on the CPU: a program that
compiles the host runtime's own source with a main() of its own and links the
built library, so that the rules checked are the ones that launch."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2406_16064_amd")

HEAD = r"""
#include "%s/csrc/plan.hip"

Group group(int nx, int ny, int nz, bool pot) {
  Group G;
  G.mesh = mm_mesh{nx, ny, nz, 3e-9, 2e-9, 2.5e-9};
  G.ncomp = nz == 1 ? 4 : 6;
  if (pot) set_padded(G, pick_padded_pot(nx, true), pick_padded_pot(ny, false), pick_padded_pot(nz, false));
  else set_padded(G, pick_padded(nx, true), pick_padded(ny, false), pick_padded(nz, false));
  return G;
}
size_t csz_of(mm_precision prec) { return prec == MM_F32 ? sizeof(Cx<float>) : sizeof(Cx<double>); }
""" % PKG


def _run(tmp_path, main):
    """Lines that the program with this main() prints, split into words."""
    if not os.path.exists(os.path.join(PKG, "libmmx.so")):
        pytest.fail("libmmx.so not built (run python -m paper_2406_16064_amd.build)")
    from paper_2406_16064_amd.build import _hipcc
    src, exe = str(tmp_path / "rules.hip"), str(tmp_path / "rules")
    with open(src, "w") as f:
        f.write(HEAD + main)
    r = subprocess.run([_hipcc(), "--offload-arch=gfx950", "-O0", "-std=c++17", src, "-o", exe, "-L" + PKG,
                        "-l:libmmx.so", "-Wl,-rpath," + PKG], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return [line.split() for line in r.stdout.splitlines()]


def test_potential_energy_partials_written_are_those_reserved(tmp_path):
    """Scalar-potential route: the energy pass writes one partial sum a workgroup;
    their number, by the rows the launch takes, is the one that the buffer and the
    reduction count by the launch shape, for every shape that a plan accepts."""
    lines = _run(tmp_path, r"""
int main() {
  for (mm_precision prec : {MM_F32, MM_F64})
    for (int nx : {20, 128, 256, 400, 487, 509, 512, 700, 1000, 1024})
      for (int ny : {1, 3, 9, 64, 512})
        for (int nz : {2, 16}) {
          Group G = group(nx, ny, nz, true);
          if (choose_tuning(G, prec, csz_of(prec), true) != MM_OK) continue;
          const Tuning def = G.tu;
          for (int ty : {0, 1, 2, 4, 8, 16})  // 0: the default shape
            for (int nt : {64, 128, 256, 512}) {
              Tuning t = def;
              if (ty > 0) {
                t.ty_x = ty;
                t.nt_i = nt;
                t.tpc_x = nt / (3 * ty);
                if (!tuning_ok(G, t, prec, csz_of(prec))) continue;
              }
              G.tu = t;
              if (!(prec == MM_F32 ? pot_fits<float>(G) : pot_fits<double>(G))) continue;
              const int rows = pot_x_rows(G.g, t, MODE_ENERGY);
              printf("%d %d %d %d %d %d %d %d\n", (int)prec, nx, ny, nz, ty, t.ty_x,
                     nz * ((ny + rows - 1) / rows), eval_blocks_per_inst(G.g, t));
            }
        }
}
""")
    rows = [[int(v) for v in line] for line in lines]
    for prec, nx, ny, nz, ty, ty_x, written, reserved in rows:
        assert written == reserved, (prec, nx, ny, nz, ty_x)
    # shapes of more than two rows on long compiled rows are among them, by default too
    assert any(nx in (509, 512) and ty_x > 2 for _, nx, _, _, _, ty_x, _, _ in rows)
    assert {ty_x for prec, nx, ny, nz, ty, ty_x, _, _ in rows if (prec, nx, ny, nz, ty) == (0, 512, 512, 16, 0)} == {4}


def test_compiled_inverse_x_takes_every_mesh_of_a_mixed_batch(tmp_path):
    """Batch launches: a mesh whose rows have a compiled length with threes takes the
    compiled inverse-x kernels with its own threads, one of a power of two up to
    256 points wherever the launch has 512, at most four cells a thread; the sweep's
    meshes together have 512."""
    lines = _run(tmp_path, r"""
int main() {
  for (mm_precision prec : {MM_F32, MM_F64})
    for (int nx = 2; nx <= 1024; ++nx)
      for (int ny : {1, 2, 5, 16, 64, 256})
        for (int nz : {1, 4}) {
          Group G = group(nx, ny, nz, false);
          if (!sr_compiled(G.g.Lx)) continue;
          for (int n : {1, 4, 32, 256, 4096}) {
            if (choose_tuning(G, prec, csz_of(prec), false, (long long)n * ny * nz) != MM_OK) continue;
            printf("%d %d %d %d %d %d %d %d %d\n", (int)prec, nx, ny, nz, n, G.g.Lx,
                   inv_x_any(G.g, G.tu, G.tu.nt_i) ? 1 : 0, inv_x_any(G.g, G.tu, 512) ? 1 : 0,
                   (G.tu.ty_x * nx + G.tu.nt_i - 1) / G.tu.nt_i);
          }
        }
  // launches of the sweep's sizes, films and two planes, n instances of each
  for (mm_precision prec : {MM_F32, MM_F64})
    for (int n : {4, 32}) {
      const int sizes[] = {32, 64, 96, 128, 192, 256};
      long long rows = 0;
      for (int a : sizes) rows += n * 3LL * a;
      std::vector<Group> gs;
      int nt = 64;
      for (int a : sizes)
        for (int nz : {1, 2}) {
          gs.push_back(group(a, a, nz, false));
          if (choose_tuning(gs.back(), prec, csz_of(prec), false, rows) != MM_OK) return 1;
          nt = std::max(nt, gs.back().tu.nt_i);
        }
      for (const Group& G : gs) printf("sweep %d %d %d\n", nt, G.g.nx, inv_x_any(G.g, G.tu, nt) ? 1 : 0);
    }
}
""")
    rows = [[int(v) for v in line] for line in lines if line[0] != "sweep"]
    assert len(rows) > 10000
    for prec, nx, ny, nz, n, Lx, own, with512, cells in rows:
        if Lx & (Lx - 1) or Lx <= 256:
            assert with512 and cells <= 4, (prec, nx, ny, nz, n, Lx, cells)
        if Lx & (Lx - 1):
            assert own, (prec, nx, ny, nz, n, Lx)
    sweep = [line[1:] for line in lines if line[0] == "sweep"]
    assert len(sweep) == 48 and all(takes == "1" for _, _, takes in sweep)


def test_forced_shapes_of_the_dispatch_tests_are_accepted(tmp_path):
    """The launch shapes that the GPU dispatch tests force are valid ones, so that
    none of them falls back to the default shape or is left out; shapes past the
    threads, the LDS or the rows are refused."""
    lines = _run(tmp_path, r"""
bool ok(mm_precision prec, int nx, int ny, int nz, int ty, int nt, bool pot) {
  Group G = group(nx, ny, nz, pot);
  if (choose_tuning(G, prec, csz_of(prec), pot) != MM_OK) return false;
  Tuning t = G.tu;
  if (pot) {
    t.ty_f = 1;
    t.tpc_f = t.nt_f;
  }
  t.ty_x = ty;
  t.nt_i = nt;
  t.tpc_x = nt / (3 * ty);
  if (!tuning_ok(G, t, prec, csz_of(prec))) return false;
  G.tu = t;
  return !pot || (prec == MM_F32 ? pot_fits<float>(G) : pot_fits<double>(G));
}
int main() {
  using S = std::array<int, 3>;
  for (int nx : {24, 81, 100, 128, 162, 200})
    for (S s : {S{1, 64}, S{2, 128}, S{4, 256}}) printf("taken %d\n", ok(MM_F64, nx, 6, 1, s[0], s[1], false));
  for (mm_precision prec : {MM_F32, MM_F64}) {
    for (S s : {S{128, 1}, S{127, 4}, S{256, 2}, S{512, 4}, S{512, 1}, S{509, 2}, S{1024, 2}, S{256, 8}, S{509, 4}, S{512, 2}})
      printf("taken %d\n", ok(prec, s[0], 9, 2, s[1], 512, true));
    printf("refused %d\n", ok(prec, 128, 6, 1, 8, 256, false));   // more rows than the mesh has
    printf("refused %d\n", ok(prec, 128, 6, 1, 3, 256, false));   // not a power of two
    printf("refused %d\n", ok(prec, 128, 6, 1, 4, 64, false));    // too few threads a column
    printf("refused %d\n", ok(prec, 128, 6, 1, 1, 1024, false));  // too many threads
    printf("refused %d\n", ok(prec, 1024, 9, 2, 4, 512, true));   // too few threads a column
  }
}
""")
    assert [v for k, v in lines if k == "taken"] == ["1"] * 38
    assert [v for k, v in lines if k == "refused"] == ["0"] * 10
