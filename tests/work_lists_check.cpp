// Work lists of a tree with cut rows, one mistake planted at a time: each has
// to be reported by same_work. Prints the mistakes that were not.
#include <cstdio>
#include <functional>
#include <numeric>

#include "tables.hpp"

using namespace ca;

static void insert(ChunkTree* t, int64_t sid, int shared, int own) {
  std::vector<int32_t> tok(shared + own);
  std::iota(tok.begin(), tok.begin() + shared, 0);
  std::iota(tok.begin() + shared, tok.end(), static_cast<int32_t>(100000 * (sid + 1)));
  std::vector<KvJob> jobs;
  int64_t matched = 0;
  if (t->insert(sid, tok.data(), static_cast<int64_t>(tok.size()), &jobs, &matched) != Err::ok)
    std::printf("insert failed\n");
}

int main() {
  ChunkTree tree(16, 4096);
  insert(&tree, 0, 100, 2000);  // cut, with shared chunks
  insert(&tree, 1, 100, 30);    // whole, with shared chunks
  insert(&tree, 2, 0, 1500);    // cut, nothing shared
  insert(&tree, 3, 0, 20);      // whole, written directly
  Tables T;
  build_tables(tree, &T);
  WorkLists good;
  build_work(tree, T, 2, -1, true, 4, 256, &good, false, 512);
  if (good.split_rows != 2) std::printf("split rows %d\n", good.split_rows);
  if (*same_work(good, good)) std::printf("equal lists: %s\n", same_work(good, good));
  WorkLists whole;
  build_work(tree, T, good.seg_chunks, 0, true, 4, 256, &whole, false, 512);
  if (*same_work(good, whole)) std::printf("cut against whole: %s\n", same_work(good, whole));

  auto item = [](WorkLists& w, int row, int nth) -> SfItem& {
    for (SfItem& it : w.items)
      if (it.row == row && nth-- == 0) return it;
    std::printf("no such item\n");
    return w.items[0];
  };
  int64_t row_of[4];
  for (size_t r = 0; r < T.row_seq.size(); ++r) row_of[T.row_seq[r]] = static_cast<int64_t>(r);
  const int cut = static_cast<int>(row_of[0]), kept = static_cast<int>(row_of[1]),
            alone = static_cast<int>(row_of[2]), direct = static_cast<int>(row_of[3]);
  const struct {
    const char* what;
    std::function<void(WorkLists&)> plant;
  } mistakes[] = {
      {"two pieces write one partial", [&](WorkLists& w) { item(w, cut, 1).out_part = item(w, cut, 0).out_part; }},
      {"pieces of two rows write one partial",
       [&](WorkLists& w) { item(w, cut, 0).out_part = item(w, alone, 0).out_part; }},
      {"a piece writes past the partials",
       [&](WorkLists& w) { item(w, alone, 0).out_part = static_cast<int32_t>(w.n_parts); }},
      {"too few partials counted", [&](WorkLists& w) { --w.n_parts; }},
      {"a piece's partial is not folded",
       [&](WorkLists& w) {
         w.parts.erase(w.parts.begin() + w.part_ptr[alone + 1] - 1);
         for (size_t r = alone + 1; r < w.part_ptr.size(); ++r) --w.part_ptr[r];
         fill_item_records(&w);
       }},
      {"a partial is folded twice", [&](WorkLists& w) { w.parts[w.part_ptr[cut]] = w.parts[w.part_ptr[cut] + 1]; }},
      {"pieces folded in another order",
       [&](WorkLists& w) { std::swap(w.parts[w.part_ptr[alone]], w.parts[w.part_ptr[alone] + 1]); }},
      {"a row counts a partial of its neighbour",
       [&](WorkLists& w) {
         ++w.part_ptr[cut + 1];
         fill_item_records(&w);
       }},
      {"segments folded in another order",
       [&](WorkLists& w) { std::swap(w.parts[w.part_ptr[cut]], w.parts[w.part_ptr[cut] + 1]); }},
      {"pieces overlap", [&](WorkLists& w) { ++item(w, alone, 0).ce; }},
      {"a whole row's piece writes o instead of its partial", [&](WorkLists& w) { item(w, kept, 0).out_part = -1; }},
      {"a direct row writes a partial", [&](WorkLists& w) { item(w, direct, 0).out_part = 0; }},
      {"a cut row is not merged", [&](WorkLists& w) { w.mg_rows.pop_back(); }},
      {"an item belongs to another row", [&](WorkLists& w) { item(w, direct, 0).row = kept; }},
      {"a piece is missing", [&](WorkLists& w) { w.items.pop_back(); }},
      {"a slot differs", [&](WorkLists& w) { ++w.priv_slot.back(); }},
  };
  for (const auto& m : mistakes) {
    WorkLists bad = good;
    m.plant(bad);
    if (!*same_work(bad, good)) std::printf("not found: %s\n", m.what);
    if (!*same_work(good, bad)) std::printf("not found on the other side: %s\n", m.what);
  }
  return 0;
}
