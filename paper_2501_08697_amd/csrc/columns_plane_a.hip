#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<8>(const ColumnsCall &);
template int columns_plane_n1<12>(const ColumnsCall &);
template int columns_plane_n1<16>(const ColumnsCall &);
template int columns_plane_n1<18>(const ColumnsCall &);
}  // namespace apw
