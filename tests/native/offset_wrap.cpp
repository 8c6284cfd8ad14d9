// Host offsets that run past 2^31 and come around to the stated total: every
// difference is a ligand's size modulo 2^32, yet half of the offsets are negative.
#include <cstdio>
#include <cstring>
#include <vector>

#include "host_checks.h"

int main() {
  const int n = 16900000;   // of 256 atoms: 2^32 and 31 432 704 more
  std::vector<int32_t> ao(n + 1), to(n + 1, 0), ta(2, 0);
  for (int i = 0; i <= n; ++i) ao[i] = (int32_t)(256u * (uint32_t)i);
  const int fake = 0;
  lg_ligands L;
  std::memset(&L, 0, sizeof L);
  L.n = n;
  L.total_atoms = ao[n];
  L.atom_offset = L.tors_offset = L.tors_atoms = &fake;
  L.x = L.y = L.z = L.inv_bond_len = L.ref_point = (const float*)&fake;
  L.frag_mask = (const uint32_t*)&fake;
  L.atom_offset_host = ao.data();
  L.tors_offset_host = to.data();
  L.tors_atoms_host = ta.data();
  if (L.total_atoms < n) return 2;
  if (lghost::check_ligands(&L, true) == LG_OK) {
    std::puts("offsets that wrap around were accepted");
    return 1;
  }
  L.n = 1000;   // the same offsets before any wrap are in order
  L.total_atoms = ao[1000];
  return lghost::check_ligands(&L, true) == LG_OK ? 0 : 3;
}
